// Host side of the AMS-Quant library: the offline quantizer (Sec. 3.1) and the
// packer into the gfx950 layout (Sec. 3.3 stage 1), plus the size queries.
// Compiled with -ffp-contract=off: the squared-error comparison of the adaptive
// search is specified as plain IEEE fp64 operations in member order.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <thread>
#include <type_traits>
#include <vector>

#include "../../include/ams.h"
#include "ams_layout.h"

namespace {

using ams::FormatInfo;

// ---- binary16 <-> double -------------------------------------------------
inline double half_to_double(uint16_t h) {
  int s = h >> 15, e = (h >> 10) & 31, m = h & 1023;
  double v;
  if (e == 0)
    v = std::ldexp((double)m, -24);
  else if (e == 31)
    v = m ? NAN : INFINITY;
  else
    v = std::ldexp((double)(1024 + m), e - 25);
  return s ? -v : v;
}

// round-to-nearest-even conversion of a finite non-negative double
inline uint16_t double_to_half_bits(double a) {
  if (a == 0) return 0;
  int ex;
  (void)std::frexp(a, &ex);  // a = f * 2^ex, f in [0.5, 1)
  int e = ex - 1;            // a = 1.xxx * 2^e
  if (e < -14) e = -14;      // subnormal quantum 2^-24
  double q = std::nearbyint(std::ldexp(a, 10 - e));  // integer significand, RNE
  if (q >= 2048) {           // rounded up into the next binade
    q = 1024;
    e += 1;
  }
  if (e > 15) return 0x7C00;  // overflow to inf (cannot happen for absmax / Fmax)
  if (q < 1024) return (uint16_t)q;  // subnormal (or zero)
  return (uint16_t)(((e + 15) << 10) | ((int)q - 1024));
}

// ---- Sec. 2.2: magnitude of a magnitude code, bias 1 ----------------------
struct Magnitudes {
  double v[4][32];  // [mantissa bits][code]
  Magnitudes() {
    for (int mbits = 0; mbits < 4; mbits++)
      for (int c = 0; c < 32; c++) {
        const int e = c >> mbits, m = c & ((1 << mbits) - 1);
        v[mbits][c] = e == 0 ? std::ldexp((double)m, -mbits) : std::ldexp((double)((1 << mbits) + m), e - 1 - mbits);
      }
  }
};
const Magnitudes g_magnitudes;
inline double magnitude(int mag_code, int mbits) { return g_magnitudes.v[mbits][mag_code]; }

// Round half to even of 0 <= x < 2^51: adding 1.5 * 2^52 leaves no bits below the units.
inline double round_even(double x) { return (x + 0x1.8p52) - 0x1.8p52; }

// ---- Eq. 1: Round(t) = nearest magnitude, ties to the even code, saturating
inline int rtn_magnitude_code(double a, int mbits) {
  // the grid is uniform with step 2^-m below 2, 2^(1-m) in [2,4), 2^(2-m) from 4 on
  const int one = 1 << mbits;  // code of 1.0
  if (a < 2.0) return (int)round_even(a * one);                                  // 0 .. 2*one
  if (a < 4.0) return std::min(one + (int)round_even(a * (one * 0.5)), 4 * one - 1);  // one + (one .. 2*one)
  if (a >= 16.0) return 4 * one - 1;
  return std::min(2 * one + (int)round_even(a * (one * 0.25)), 4 * one - 1);
}

// Re-rounding variant of the search (not in the paper): nearest magnitude among the codes
// that end in m0.  The candidates are walked in order; an exact tie between two
// neighbours goes to the one whose upper part (code >> 1) is even; inputs above the
// largest candidate land on it.
inline int reround_magnitude_code(double a, int mbits, int m0) {
  const int n_upper = 2 << mbits;  // 4 * 2^mbits magnitude codes, every other one
  int best = 0;
  double best_d = std::fabs(a - magnitude(m0, mbits));
  for (int j = 1; j < n_upper; j++) {
    const double d = std::fabs(a - magnitude(2 * j + m0, mbits));
    if (d > best_d) break;  // the magnitudes ascend: from here on they are further and further away
    if (d < best_d || (j & 1) == 0) best = j, best_d = d;
  }
  return 2 * best + m0;
}

struct WideRow;
struct RowQuant {
  int fmt, mbits, group;
  double fmax;
  int search;  // AMS_SEARCH_*
  const WideRow* vectors;  // the instruction set's vector path (nullptr: none)
};

// Largest magnitude of a run of weights as binary16 bits (they order like the magnitudes); 0x7C00 or more when one of
// them is inf or NaN.
uint16_t abs_max_bits(const uint16_t* w, int64_t K) {
  uint16_t m = 0;
  for (int64_t k = 0; k < K; k++) m = std::max<uint16_t>(m, w[k] & 0x7FFF);
  return m;
}

// Eq. 1: the fp16 scale for a given largest magnitude (1.0 where it would be zero)
uint16_t scale_bits(uint16_t absmax, double fmax) {
  const uint16_t sb = double_to_half_bits(half_to_double(absmax) / fmax);
  return sb == 0 ? (uint16_t)0x3C00 : sb;
}

// The two candidate magnitude codes (shared bit 0 and 1) of a weight of magnitude aw.
inline void candidates(const RowQuant& q, double aw, double s, int (&c)[2]) {
  const double a = aw / s;
  if (q.search == AMS_SEARCH_REROUND) {
    c[0] = reround_magnitude_code(a, q.mbits, 0);
    c[1] = reround_magnitude_code(a, q.mbits, 1);
  } else {  // Sec. 3.1: the RTN code with its last bit set to m0
    const int mc = rtn_magnitude_code(a, q.mbits);
    c[0] = mc & ~1;
    c[1] = mc | 1;
  }
}

typedef double d2 __attribute__((vector_size(16)));

// |w| of a finite binary16 magnitude, exact and whatever the thread's denormal mode: the fields of a normal one moved
// into binary64's, a subnormal one counted in units of 2^-24.
inline double abs_to_double(uint16_t mag) {
  if (mag < 0x400) return mag * 0x1p-24;
  const uint64_t bits = ((uint64_t)mag << 42) + ((uint64_t)(1023 - 15) << 52);
  double d;
  std::memcpy(&d, &bits, 8);
  return d;
}

// What quantizing a weight needs to know of its magnitude, for one scale.  The candidate codes are step functions of
// |w| (division, rounding and the search are monotone), so the magnitudes fall into at most 64 intervals with one pair
// of codes each; `interval` has an entry per binary16 magnitude up to the row's largest.
struct Steps {
  std::vector<uint8_t> interval;
  int n = 0;
  uint8_t code[2][64];  // candidate codes
  d2 value[64];         // their magnitudes times the scale (Eq. 2)

  void add(const RowQuant& q, double s, const int (&c)[2]) {
    code[0][n] = (uint8_t)c[0], code[1][n] = (uint8_t)c[1];
    value[n] = d2{magnitude(c[0], q.mbits) * s, magnitude(c[1], q.mbits) * s};
    n++;
  }
  // All magnitudes 0 .. top.
  void build(const RowQuant& q, double s, uint16_t top) {
    if (interval.size() <= top) interval.resize((size_t)top + 1);
    n = 0;
    int lo = 0, cl[2];
    candidates(q, 0.0, s, cl);
    add(q, s, cl);
    int ch[2];
    candidates(q, abs_to_double(top), s, ch);
    while (cl[0] != ch[0] || cl[1] != ch[1]) {  // the first magnitude in (lo, top] with other codes than lo's
      int a = lo, b = top, c[2], cb[2] = {ch[0], ch[1]};
      while (b - a > 1) {
        const int mid = (a + b) / 2;
        candidates(q, abs_to_double((uint16_t)mid), s, c);
        if (c[0] == cl[0] && c[1] == cl[1])
          a = mid;
        else
          b = mid, cb[0] = c[0], cb[1] = c[1];
      }
      std::memset(interval.data() + lo, n - 1, (size_t)(b - lo));
      lo = b;
      cl[0] = cb[0], cl[1] = cb[1];
      add(q, s, cl);
    }
    std::memset(interval.data() + lo, n - 1, (size_t)top + 1 - lo);
  }
};

// ---- many groups at a time ----------------------------------------------------
// The quantizer of Sec. 3.1 on vectors of L groups (16 with AVX-512, 8 with AVX2): lane g of member vector p is weight p
// of group g.  The codes are the ones of candidates() and of the search in quantize_row, bit for bit: what is decided in
// binary32 is decided again in binary64, with their operations in their order, wherever the first decision is closer than
// its error allows.  Plain vector arithmetic, compiled for both instruction sets and called where the processor has them.
// Bound by vector arithmetic (about 50 operations per member vector).  A strip of 16 x 4096 FP5.33 weights on one core of an EPYC with
// AVX-512: quantized and packed 92 -> 32 us (codes looked up and placed by table -> wide_records), FP6, codes then table, 109 -> 50.
#define AMS_INLINE __attribute__((always_inline)) inline
template <class T, int L>
using Vec = T __attribute__((ext_vector_type(L)));

template <class V>
AMS_INLINE V load_vec(const void* p) {
  V v;
  std::memcpy(&v, p, sizeof(v));
  return v;
}

// Members 0 .. G-1 of L groups of G neighbouring weights.
template <int G, int L>
AMS_INLINE void load_members(const uint16_t* w, Vec<uint16_t, L> (&m)[G]) {
  if constexpr (G == 1) {
    m[0] = load_vec<Vec<uint16_t, L>>(w);
  } else {
    constexpr int HALF = G == 2 ? L : 2 * L;  // weights of the first of the two vectors that are shuffled
    typedef Vec<uint16_t, HALF> V;
    const V a = load_vec<V>(w);
    V b = 0;
    std::memcpy(&b, w + HALF, (G * L - HALF) * 2);
#define AMS_PICK8(p, o) (o) * G + p, (o + 1) * G + p, (o + 2) * G + p, (o + 3) * G + p, (o + 4) * G + p, (o + 5) * G + p, (o + 6) * G + p, (o + 7) * G + p
#define AMS_PICK(p)                                                              \
  if constexpr (p < G) {                                                         \
    if constexpr (L == 8)                                                        \
      m[p < G ? p : 0] = __builtin_shufflevector(a, b, AMS_PICK8(p, 0));                  \
    else                                                                         \
      m[p < G ? p : 0] = __builtin_shufflevector(a, b, AMS_PICK8(p, 0), AMS_PICK8(p, 8)); \
  }
    AMS_PICK(0) AMS_PICK(1) AMS_PICK(2) AMS_PICK(3)
#undef AMS_PICK
#undef AMS_PICK8
  }
}

// Codes without their last bit (the candidates with shared bit 0) and the chosen last bit of L groups, in binary64.
template <int G, int L, int MBITS>
AMS_INLINE void quantize_groups_exactly(const Vec<uint16_t, L> (&w)[G], double s, Vec<int32_t, L> (&upper)[G], Vec<int32_t, L>& last) {
  typedef Vec<double, L> D;
  constexpr double one = 1 << MBITS;  // code of 1.0
  D sse0 = 0, sse1 = 0;
#pragma unroll
  for (int p = 0; p < G; p++) {
    const Vec<uint16_t, L> mag = w[p] & (uint16_t)0x7FFF;
    const D aw = __builtin_convertvector(__builtin_convertvector(__builtin_bit_cast(Vec<_Float16, L>, mag), Vec<float, L>), D);
    const D a = aw / s;
    // the grid is uniform below 2, in [2, 4) and from 4 on (rtn_magnitude_code)
    const D scale = a < 2.0 ? (D)one : (a < 4.0 ? (D)(one * 0.5) : (D)(one * 0.25));
    const D first = a < 2.0 ? (D)0.0 : (a < 4.0 ? (D)one : (D)(2 * one));
    D code = first + ((a * scale + 0x1.8p52) - 0x1.8p52);
    code = code < 4 * one - 1 ? code : (D)(4 * one - 1);
    upper[p] = __builtin_convertvector(code, Vec<int32_t, L>) & ~1;
    // magnitudes of the candidates: both lie in one piece of the grid, neighbours a step apart
    const D c0 = __builtin_convertvector(upper[p], D);
    const D base = c0 < 2 * one ? (D)0.0 : (c0 < 3 * one ? (D)one : (D)(2 * one));
    const D step = c0 < 2 * one ? (D)(1 / one) : (c0 < 3 * one ? (D)(2 / one) : (D)(4 / one));
    const D v0 = (c0 - base) * step;
    const D d0 = v0 * s - aw, d1 = (v0 + step) * s - aw;  // Eq. 2 with last bit 0 and 1
    sse0 = sse0 + d0 * d0;
    sse1 = sse1 + d1 * d1;
  }
  last = __builtin_convertvector(sse1 < sse0, Vec<int32_t, L>) & 1;  // a tie keeps 0
}

// The same from a = |w| * rs, rs = 1 / s in binary32, which is within 2^-22 of |w| / s of its own size.
//   code: a times the inverse step is at most 16 where the code is not the largest, so it is off by 2^-18; it rounds to
//     the same integer unless it lies within 2^-16 of a half.  (Where a is on the other side of 2 or 4 than the quotient, the
//     pieces of the grid meet there and give the same code.)
//   last bit: the difference of the squared errors, in units of s^2, is the sum of step * (2 (v0 - a) + step).  A term is off
//     by step * (2^-21 a + 2^-22 step) at most, its sums' rounding by less than that: its sign holds beyond 2^-19 of the sum
//     of step * (a + step).
// The largest magnitude is 7.5 times the scale, so a above 16 means a scale that was rounded among the smallest binary16
// numbers.
template <int G, int L, int MBITS>
AMS_INLINE void quantize_groups(const Vec<uint16_t, L> (&w)[G], double s, float rs, Vec<int32_t, L> (&upper)[G], Vec<int32_t, L>& last) {
  typedef Vec<float, L> F;
  constexpr float one = 1 << MBITS;
  F diff = 0, size = 0, nearest = 0, largest = 0;
#pragma unroll
  for (int p = 0; p < G; p++) {
    const Vec<uint16_t, L> mag = w[p] & (uint16_t)0x7FFF;
    const F a = __builtin_convertvector(__builtin_bit_cast(Vec<_Float16, L>, mag), F) * rs;
    const F scale = a < 2.0f ? (F)one : (a < 4.0f ? (F)(one * 0.5f) : (F)(one * 0.25f));
    const F first = a < 2.0f ? (F)0.0f : (a < 4.0f ? (F)one : (F)(2 * one));
    const F x = a * scale, r = __builtin_elementwise_roundeven(x);
    nearest = __builtin_elementwise_max(nearest, __builtin_elementwise_abs(x - r));
    largest = __builtin_elementwise_max(largest, a);
    const F code = __builtin_elementwise_min(first + r, (F)(4 * one - 1));
    upper[p] = __builtin_convertvector(code, Vec<int32_t, L>) & ~1;
    const F c0 = __builtin_convertvector(upper[p], F);
    const F base = c0 < 2 * one ? (F)0.0f : (c0 < 3 * one ? (F)one : (F)(2 * one));
    const F step = c0 < 2 * one ? (F)(1 / one) : (c0 < 3 * one ? (F)(2 / one) : (F)(4 / one));
    const F d0 = (c0 - base) * step - a;
    diff = diff + step * (d0 + d0 + step);
    size = size + step * (a + step);
  }
  last = (diff < 0.0f) & 1;
  if (__builtin_reduce_or((nearest > 0.5f - 0x1p-16f) | (largest > 16.0f) | (__builtin_elementwise_abs(diff) <= size * 0x1p-19f)))
    quantize_groups_exactly<G, L, MBITS>(w, s, upper, last);
}

// 1 where a weight is negative (not of -0)
template <int L>
AMS_INLINE Vec<int32_t, L> sign_of(const Vec<uint16_t, L>& w) {
  return (__builtin_convertvector(w, Vec<int32_t, L>) > 0x8000) & 1;
}

// Whole vectors of L groups of a row (or run) from weight k on, as codes; returns where they end.
template <int G, int L, int MBITS>
AMS_INLINE int64_t wide_codes(const uint16_t* w, int64_t k, int64_t K, double s, float rs, uint8_t* codes) {
  for (; k + L * G <= K; k += L * G) {
    Vec<uint16_t, L> m[G];
    Vec<int32_t, L> upper[G], last;
    load_members<G, L>(w + k, m);
    quantize_groups<G, L, MBITS>(m, s, rs, upper, last);
    uint8_t c[G][L];
#pragma unroll
    for (int p = 0; p < G; p++) {
      const Vec<uint8_t, L> v = __builtin_convertvector(upper[p] | last | sign_of<L>(m[p]) << (2 + MBITS), Vec<uint8_t, L>);
      if constexpr (G == 1)
        std::memcpy(codes + k, &v, L);
      else
        std::memcpy(c[p], &v, L);
    }
    if constexpr (G > 1) {
      for (int g = 0; g < L; g++)
        for (int p = 0; p < G; p++) codes[k + g * G + p] = c[p][g];
    }
  }
  return k;
}

// Whole records of row r of strip t, straight into the packed matrix, for the two formats whose half-words are whole
// sharing groups; w points at the row's record `rec`.
template <int FMT, int L>
AMS_INLINE void wide_records(const uint16_t* w, int64_t rec, int64_t rec_end, double s, uint8_t* packed, int64_t n_strips, int64_t t, int r) {
  static_assert(FMT == ams::kFmtFp533 || FMT == ams::kFmtFp425, "half-words that are groups");
  constexpr FormatInfo fi = ams::kFormats[FMT];
  constexpr int G = fi.group, MBITS = fi.code_bits - 3;
  const float rs = 1.0f / (float)s;
  for (; rec < rec_end; rec++, w += fi.rec_k) {
    const ams::RecordPlace rp = ams::record_place(fi, n_strips, t, rec);
    for (int h0 = 0; h0 < 32; h0 += L) {  // half-words of the record: eight to a lane chunk
      Vec<uint16_t, L> m[G];
      Vec<int32_t, L> upper[G], last;
      load_members<G, L>(w + h0 * G, m);
      quantize_groups<G, L, MBITS>(m, s, rs, upper, last);
      Vec<int32_t, L> hw = FMT == ams::kFmtFp533 ? last << 12 : (Vec<int32_t, L>)0;
#pragma unroll
      for (int p = 0; p < G; p++) {
        constexpr int sign_at[2][4] = {{15, 12, 14, 13}, {15, 14, 13, 0}};
        hw |= sign_of<L>(m[p]) << sign_at[FMT == ams::kFmtFp533][p] | (upper[p] >> 1) << (FMT == ams::kFmtFp533 ? 8 - 4 * p : 9 - 3 * p);
      }
      const Vec<uint16_t, L> out = __builtin_convertvector(hw, Vec<uint16_t, L>);
      uint32_t bits = 0;  // FP4.25: the groups' last bits, one per half-word
      if constexpr (FMT == ams::kFmtFp425) {
        Vec<int32_t, L> at;
#pragma unroll
        for (int x = 0; x < L; x++) at[x] = x / 8 * 8 + 4 * (x & 1) + (x & 7) / 2;  // of half-word 2d + h: bit 4h + d of its chunk's byte
        bits = (uint32_t)__builtin_reduce_or(last << at);
      }
#pragma unroll
      for (int c = 0; c < L / 8; c++) {
        const int lane = (h0 / 8 + c) * 16 + r;
        std::memcpy(packed + rp.chunks + lane * 16, (const uint8_t*)&out + 16 * c, 16);
        if constexpr (FMT == ams::kFmtFp425) packed[rp.side + 4 * lane + rp.side_shift / 8] = (uint8_t)(bits >> (8 * c));
      }
    }
  }
}

// One row (or run) in one format, for one instruction set.
struct WideRow {
  int lanes;
  int64_t (*codes)(int fmt, const uint16_t* w, int64_t K, double s, uint8_t* codes);
  void (*records)(int fmt, const uint16_t* w, int64_t rec, int64_t rec_end, double s, uint8_t* packed, int64_t n_strips, int64_t t, int r);
};
template <int L>
AMS_INLINE int64_t wide_codes_of(int fmt, const uint16_t* w, int64_t k, int64_t K, double s, uint8_t* codes) {
  const float rs = 1.0f / (float)s;
  switch (fmt) {
    case ams::kFmtFp533: return wide_codes<3, L, 3>(w, k, K, s, rs, codes);
    case ams::kFmtFp425: return wide_codes<4, L, 2>(w, k, K, s, rs, codes);
    case ams::kFmtFp45: return wide_codes<2, L, 2>(w, k, K, s, rs, codes);
    case ams::kFmtFp433: return wide_codes<3, L, 2>(w, k, K, s, rs, codes);
    case ams::kFmtFp6: return wide_codes<1, L, 3>(w, k, K, s, rs, codes);
    case ams::kFmtFp5: return wide_codes<1, L, 2>(w, k, K, s, rs, codes);
    default: return wide_codes<1, L, 1>(w, k, K, s, rs, codes);
  }
}
template <int L>
AMS_INLINE void wide_records_of(int fmt, const uint16_t* w, int64_t rec, int64_t rec_end, double s, uint8_t* packed, int64_t n_strips, int64_t t, int r) {
  if (fmt == ams::kFmtFp533)
    wide_records<ams::kFmtFp533, L>(w, rec, rec_end, s, packed, n_strips, t, r);
  else
    wide_records<ams::kFmtFp425, L>(w, rec, rec_end, s, packed, n_strips, t, r);
}
#define AMS_AVX512 __attribute__((target("avx512f,avx512bw,avx512dq,avx512vl,f16c")))
#define AMS_AVX2 __attribute__((target("avx2,f16c")))
AMS_AVX512 int64_t codes_avx512(int fmt, const uint16_t* w, int64_t K, double s, uint8_t* codes) {
  return wide_codes_of<8>(fmt, w, wide_codes_of<16>(fmt, w, 0, K, s, codes), K, s, codes);
}
AMS_AVX2 int64_t codes_avx2(int fmt, const uint16_t* w, int64_t K, double s, uint8_t* codes) { return wide_codes_of<8>(fmt, w, 0, K, s, codes); }
AMS_AVX512 void records_avx512(int fmt, const uint16_t* w, int64_t rec, int64_t rec_end, double s, uint8_t* packed, int64_t n_strips, int64_t t, int r) {
  wide_records_of<16>(fmt, w, rec, rec_end, s, packed, n_strips, t, r);
}
AMS_AVX2 void records_avx2(int fmt, const uint16_t* w, int64_t rec, int64_t rec_end, double s, uint8_t* packed, int64_t n_strips, int64_t t, int r) {
  wide_records_of<8>(fmt, w, rec, rec_end, s, packed, n_strips, t, r);
}
// Vectors of at most `lanes` groups: the widest that this processor has (nullptr: none; the codes are then looked up).
constexpr int kWidest = 16;
const WideRow* wide_row(int lanes) {
  static const WideRow avx512 = {16, codes_avx512, records_avx512}, avx2 = {8, codes_avx2, records_avx2};
  static const bool has512 = __builtin_cpu_supports("avx512f") && __builtin_cpu_supports("avx512bw") && __builtin_cpu_supports("avx512dq") &&
                             __builtin_cpu_supports("avx512vl") && __builtin_cpu_supports("f16c");
  static const bool has2 = __builtin_cpu_supports("avx2") && __builtin_cpu_supports("f16c");
  return lanes >= 16 && has512 ? &avx512 : lanes >= 8 && has2 ? &avx2 : nullptr;
}

// Quantize one row (or run): scale (Eq. 1), RTN, adaptive search of each group's shared bit.  Returns false on inf/NaN.
// forced_scale: 0 = the row's own scale (Eq. 1 per output channel), else the fp16 bits to use (whoever gives them has seen
// that the weights are finite).
// 4096 x 4096 FP5.33, packing included, on 16 threads: 0.9 ms in vectors, 2.2 ms with the codes looked up (the re-rounding
// search, processors without AVX2), 36 ms when every weight was divided, rounded and compared by itself with library calls.
bool quantize_row(const RowQuant& q, const uint16_t* w, int64_t K, uint8_t* codes, uint16_t* scale_out, Steps& steps, uint16_t forced_scale = 0) {
  const int sign_shift = 2 + q.mbits;
  // Looking codes up pays from about 200 weights per scale on (finding the intervals takes as long as evaluating that
  // many): 3971 x 400 FP5.33 3.3 -> 2.0 ms on 8 threads, 8000 x 200 3.5 -> 3.3, 16384 x 128 4.8 -> 5.9.
  const WideRow* const wide = q.search == AMS_SEARCH_SET_BIT && K >= 8 * q.group ? q.vectors : nullptr;  // not for less than a vector
  const bool lookup = !wide && K >= 192;
  const uint16_t absmax = !forced_scale || lookup ? abs_max_bits(w, K) : 0;
  if (absmax >= 0x7C00) return false;
  const uint16_t sb = forced_scale ? forced_scale : scale_bits(absmax, q.fmax);
  *scale_out = sb;
  const double s = half_to_double(sb);
  if (lookup) steps.build(q, s, absmax);
  auto finish = [&](int64_t k, int mag_code) {
    const uint16_t wk = w[k];
    codes[k] = (uint8_t)(mag_code | ((wk > 0x8000 ? 1 : 0) << sign_shift));  // sign bit = (w < 0): not of -0
  };
  auto groups = [&](auto group_c) {
    constexpr int G = decltype(group_c)::value;
    int64_t k0 = 0;
    if (wide) k0 = wide->codes(q.fmt, w, K, s, codes);
    if (lookup) {
      for (; k0 + G <= K; k0 += G) {
        int iv[G];
        d2 sse = {0, 0};
        for (int i = 0; i < G; i++) {
          const uint16_t mag = w[k0 + i] & 0x7FFF;
          iv[i] = steps.interval[mag];
          const double aw = abs_to_double(mag);
          const d2 d = steps.value[iv[i]] - d2{aw, aw};
          sse = sse + d * d;
        }
        const uint8_t* c = steps.code[sse[1] < sse[0] ? 1 : 0];  // a tie keeps 0
        for (int i = 0; i < G; i++) finish(k0 + i, c[iv[i]]);
      }
    }
    for (; k0 < K; k0 += G) {
      const int n = (int)std::min<int64_t>(G, K - k0);
      int c[4][2];
      double sse0 = 0, sse1 = 0;
      for (int i = 0; i < n; i++) {
        const double aw = abs_to_double(w[k0 + i] & 0x7FFF);
        candidates(q, aw, s, c[i]);
        const double d0 = magnitude(c[i][0], q.mbits) * s - aw;  // Eq. 2 with last bit 0
        const double d1 = magnitude(c[i][1], q.mbits) * s - aw;  // ... with last bit 1
        sse0 = sse0 + d0 * d0;
        sse1 = sse1 + d1 * d1;
      }
      const int m0 = sse1 < sse0 ? 1 : 0;
      for (int i = 0; i < n; i++) finish(k0 + i, c[i][m0]);
    }
  };
  switch (q.group) {
    case 1: groups(std::integral_constant<int, 1>{}); break;
    case 2: groups(std::integral_constant<int, 2>{}); break;
    case 3: groups(std::integral_constant<int, 3>{}); break;
    default: groups(std::integral_constant<int, 4>{}); break;
  }
  return true;
}

// ---- layout ---------------------------------------------------------------
inline bool is_e2m3(int fmt) { return fmt == ams::kFmtFp533 || fmt == ams::kFmtFp6; }

// Bit positions of member i's sign and magnitude inside a half-word, and the bit
// (or -1) of the half-word that holds a last mantissa bit.
inline int sign_pos(int fmt, int i) {
  if (is_e2m3(fmt)) return 15 - i;
  constexpr int pos[4] = {15, 12, 14, 13};
  return pos[i];
}
inline int mag_pos(int fmt, int i) { return is_e2m3(fmt) ? 8 - 4 * i : 9 - 3 * i; }

// What one code adds to its lane chunk: the low half to the 32-bit word of its place, the high half to the side bits.
template <int FMT>
struct PlaceTable {
  uint64_t add[ams::kFormats[FMT].lane_k][64];  // [weight of the lane chunk][code]
  PlaceTable() {
    constexpr FormatInfo fi = ams::kFormats[FMT];
    // FP4-e2m1 has no last bit beside its remainder: the nibble is the whole code
    constexpr bool whole = FMT == ams::kFmtFp4;
    constexpr int mag_bits = whole ? fi.code_bits - 1 : fi.code_bits - 2;  // bits of a remainder without its sign
    for (int q = 0; q < fi.lane_k; q++)
      for (int c = 0; c < 64; c++) {
        add[q][c] = 0;
        if (c >> fi.code_bits) continue;
        const ams::Place p = ams::place(FMT, q);
        const uint32_t rem = whole ? (uint32_t)c : (uint32_t)c >> 1, lsb = whole ? 0u : (uint32_t)c & 1;
        uint32_t hw = (rem >> mag_bits) << sign_pos(FMT, p.i) | (rem & ((1u << mag_bits) - 1)) << mag_pos(FMT, p.i);
        const int sb = ams::side_bit(FMT, q);
        if (sb < 0) hw |= lsb << 12;
        add[q][c] = (uint64_t)(hw << (16 * p.h)) | (sb >= 0 ? (uint64_t)lsb << (32 + sb) : 0);
      }
  }
};

// Writes the records of strip t of a packed matrix of n_strips strips, from record `first` on.  codes: 16 rows of their K - first *
// rec_k codes (row pointer NULL = padding row).  Records beyond K that pad the last side group hold zero codes.
template <int FMT>
void pack_strip_of(const uint8_t* const rows[16], int64_t K, uint8_t* packed, int64_t n_strips, int64_t t, int64_t first) {
  static const PlaceTable<FMT> table;
  constexpr FormatInfo fi = ams::kFormats[FMT];
  const int64_t n_rec = ams::round_up(ams::round_up(K, fi.rec_k) / fi.rec_k, ams::side_group(fi));
  K -= first * fi.rec_k;
  for (int64_t j = first; j < n_rec; j++) {
    const ams::RecordPlace rp = ams::record_place(fi, n_strips, t, j);
    for (int l = 0; l < ams::kLanes; l++) {
      const uint8_t* row = rows[l & 15];
      const int64_t kbase = (j - first) * fi.rec_k + (int64_t)(l >> 4) * fi.lane_k;
      uint64_t words[4] = {0, 0, 0, 0};
      if (row && kbase + fi.lane_k <= K) {
#pragma unroll
        for (int q = 0; q < fi.lane_k; q++) words[ams::place(FMT, q).d] |= table.add[q][row[kbase + q] & 63];
      } else if (row) {  // the rest is padding: code 0 adds nothing
        for (int q = 0; q < fi.lane_k && kbase + q < K; q++) words[ams::place(FMT, q).d] |= table.add[q][row[kbase + q] & 63];
      }
      uint32_t chunk[4];
      for (int d = 0; d < 4; d++) chunk[d] = (uint32_t)words[d];
      std::memcpy(packed + rp.chunks + l * fi.chunk_bytes, chunk, (size_t)fi.chunk_bytes);
      // this record's bytes of the lane's side dword (little-endian); the other records of the group write theirs
      const uint32_t side = (uint32_t)((words[0] | words[1] | words[2] | words[3]) >> 32);
      for (int b = 0; b < fi.side_bytes; b++) packed[rp.side + 4 * l + rp.side_shift / 8 + b] = (uint8_t)(side >> (8 * b));
    }
  }
}

void pack_strip(int fmt, const uint8_t* const rows[16], int64_t K, uint8_t* packed, int64_t n_strips, int64_t t, int64_t first = 0) {
  switch (fmt) {
    case ams::kFmtFp533: return pack_strip_of<ams::kFmtFp533>(rows, K, packed, n_strips, t, first);
    case ams::kFmtFp425: return pack_strip_of<ams::kFmtFp425>(rows, K, packed, n_strips, t, first);
    case ams::kFmtFp45: return pack_strip_of<ams::kFmtFp45>(rows, K, packed, n_strips, t, first);
    case ams::kFmtFp433: return pack_strip_of<ams::kFmtFp433>(rows, K, packed, n_strips, t, first);
    case ams::kFmtFp6: return pack_strip_of<ams::kFmtFp6>(rows, K, packed, n_strips, t, first);
    case ams::kFmtFp5: return pack_strip_of<ams::kFmtFp5>(rows, K, packed, n_strips, t, first);
    default: return pack_strip_of<ams::kFmtFp4>(rows, K, packed, n_strips, t, first);
  }
}

// Strip t quantized and packed in one pass over its weights, where the format's half-words are whole sharing groups: whole
// records straight into the packed matrix, the rest of the rows and the padding as codes.  run: weights per scale (K, or a
// multiple of the record).  scale_of(r, j): where run j of row r keeps its scale.  Returns false on inf/NaN; a run that holds one
// gets zero codes and its scale is left alone, as where the codes are made first.
template <class ScaleOf>
bool quantize_and_pack_strip(const RowQuant& q, const FormatInfo& fi, const WideRow& wide, const uint16_t* W, int64_t N, int64_t K, int64_t ldw, int64_t run,
                             uint16_t forced_scale, uint8_t* packed, int64_t n_strips, int64_t t, Steps& steps, ScaleOf&& scale_of) {
  const int64_t whole = K / fi.rec_k, rest = K - whole * fi.rec_k;
  uint8_t rest_codes[16][128];
  const uint8_t* rows[16];
  bool finite = true;
  for (int r = 0; r < 16; r++) {
    const int64_t n = t * 16 + r;
    rows[r] = n < N ? rest_codes[r] : nullptr;
    auto zero_codes = [&](int64_t rec, int64_t rec_end) {  // whole records of this row
      for (; rec < rec_end; rec++) {
        const ams::RecordPlace rp = ams::record_place(fi, n_strips, t, rec);
        for (int c = 0; c < 4; c++) {
          std::memset(packed + rp.chunks + (c * 16 + r) * fi.chunk_bytes, 0, (size_t)fi.chunk_bytes);
          std::memset(packed + rp.side + 4 * (c * 16 + r) + rp.side_shift / 8, 0, (size_t)fi.side_bytes);
        }
      }
    };
    if (n >= N) {
      zero_codes(0, whole);
      continue;
    }
    const uint16_t* w = W + n * ldw;
    for (int64_t a = 0, j = 0; a < K; a += run, j++) {
      const int64_t end = std::min(K, a + run), rec = a / fi.rec_k, rec_end = std::min(end / fi.rec_k, whole);
      const uint16_t absmax = abs_max_bits(w + a, end - a);
      if (absmax >= 0x7C00) {
        finite = false;
        zero_codes(rec, rec_end);
        if (end > whole * fi.rec_k) std::memset(rest_codes[r], 0, (size_t)rest);
        continue;
      }
      const uint16_t sb = forced_scale ? forced_scale : scale_bits(absmax, q.fmax);
      *scale_of(r, j) = sb;
      wide.records(q.fmt, w + a, rec, rec_end, half_to_double(sb), packed, n_strips, t, r);
      uint16_t same;
      if (end > whole * fi.rec_k) quantize_row(q, w + whole * fi.rec_k, rest, rest_codes[r], &same, steps, sb);
    }
  }
  pack_strip(q.fmt, rows, K, packed, n_strips, t, whole);
  return finite;
}

void unpack_strip(int fmt, const FormatInfo& fi, const uint8_t* packed, int64_t n_strips, int64_t t, int64_t K, uint8_t* const rows[16]) {
  const int64_t n_rec = ams::round_up(K, fi.rec_k) / fi.rec_k;
  const bool whole = fmt == ams::kFmtFp4;
  const int mag_bits = whole ? fi.code_bits - 1 : fi.code_bits - 2;
  for (int64_t j = 0; j < n_rec; j++) {
    const ams::RecordPlace rp = ams::record_place(fi, n_strips, t, j);
    for (int l = 0; l < ams::kLanes; l++) {
      uint8_t* row = rows[l & 15];
      if (!row) continue;
      const int64_t kbase = j * fi.rec_k + (int64_t)(l >> 4) * fi.lane_k;
      uint32_t words[4] = {0, 0, 0, 0};
      std::memcpy(words, packed + rp.chunks + l * fi.chunk_bytes, (size_t)fi.chunk_bytes);
      uint32_t side = 0;
      for (int b = 0; b < fi.side_bytes; b++) side |= (uint32_t)packed[rp.side + 4 * l + rp.side_shift / 8 + b] << (8 * b);
      for (int q = 0; q < fi.lane_k; q++) {
        if (kbase + q >= K) continue;
        const ams::Place p = ams::place(fmt, q);
        const uint32_t hw = (words[p.d] >> (16 * p.h)) & 0xFFFF;
        const uint32_t rem = ((hw >> sign_pos(fmt, p.i)) & 1) << mag_bits | ((hw >> mag_pos(fmt, p.i)) & ((1u << mag_bits) - 1));
        const int sb = ams::side_bit(fmt, q);
        const uint32_t lsb = sb >= 0 ? (side >> sb) & 1 : (hw >> 12) & 1;
        row[kbase + q] = whole ? (uint8_t)rem : (uint8_t)(rem << 1 | lsb);
      }
    }
  }
}

// Whether strips are quantized and packed in one pass: nobody asks for the codes, the rows have whole records, and the format
// and the processor allow it.
const WideRow* one_pass(const RowQuant& q, const FormatInfo& fi, int64_t K, const uint8_t* codes_out) {
  const bool fits = (q.fmt == ams::kFmtFp533 || q.fmt == ams::kFmtFp425) && q.search == AMS_SEARCH_SET_BIT && !codes_out && K >= fi.rec_k;
  return fits ? q.vectors : nullptr;
}

// Time of N rows of K weights in the packer with `run` weights per scale, on one thread: every scale, and a weight in one pass,
// with the codes apart, looked up (long runs), one by one.  (Long rows are faster; on those all threads start anyway.)
double quantize_ns(const RowQuant& q, const WideRow* in_one_pass, int64_t N, int64_t K, int64_t run) {
  run = std::min(run, K);
  const bool wide = q.search == AMS_SEARCH_SET_BIT && run >= 8 * q.group && q.vectors;
  const double weight = q.search == AMS_SEARCH_REROUND ? 30 : in_one_pass ? 0.4 : wide ? 0.8 : run >= 192 ? 6 : 15;
  return N * ((K + run - 1) / run * (wide ? 30.0 : 100.0) + K * weight);
}
// The same of codes that are given: placed by table, and read back bit by bit (at a twentieth of this, four threads
// where eight pay, 256 x 768 took 620 us instead of 410).
constexpr double kPackCodesNs = 0.5, kUnpackNs = 8;

int check_shape(int fmt, int64_t N, int64_t K) {
  if (!ams::format_info(fmt)) return AMS_ERR_FORMAT;
  if (N <= 0 || K <= 0 || N > (int64_t)1 << 24 || K > (int64_t)1 << 24) return AMS_ERR_SHAPE;
  return AMS_OK;
}

// Runs body(0 .. n-1) on up to 16 threads.  False when a body threw (the only thing these bodies can
// throw is std::bad_alloc from their row buffers); a thread that cannot be started just means fewer workers.
// ns: what the whole work takes one thread.  Starting a thread costs the starter about 12 us, so the sum of both is
// least with the square root of work / 10 us: 256 x 4096 weights, 0.5 ms of work, 142 us on 7 or 8 threads, 229 on sixteen.
// (Threads that start threads in turn: 168 and 273 us.)  Below 60 us a thread comes too late to help (64 x 512 FP5.33 75 us on two
// threads, 44 on one).
template <class F>
bool parallel_for(int64_t n, double ns, F&& body) {
  unsigned hw = std::thread::hardware_concurrency();
  const int64_t worth = ns < 60e3 ? 1 : (int64_t)std::ceil(std::sqrt(ns / 10e3));
  int64_t nt = std::max<int64_t>(1, std::min<int64_t>({(int64_t)(hw ? hw : 1), (int64_t)16, n, worth}));
  struct alignas(64) Shared {  // alone on its cache line: every claim of an index takes the line away from all threads
    std::atomic<int64_t> next{0};
    std::atomic<int> failed{0};
  } shared;
  std::atomic<int64_t>& next = shared.next;
  std::atomic<int>& failed = shared.failed;
  // Every thread has a copy of the body and, the bodies capturing by value, of what it reads: on the stack of the calling thread,
  // which works on it too, the same lines were taken from one thread by another for every row (4096 x 4096 FP4.25 on 16 threads
  // 667 us, by reference 675 to 807, as the compiler happened to place things).
  auto work = [&, body] {
    try {
      for (int64_t i; !failed.load() && (i = next.fetch_add(1)) < n;) body(i);
    } catch (...) {
      failed.store(1);
    }
  };
  std::vector<std::thread> th;
  try {
    th.reserve((size_t)nt);
    for (int64_t t = 1; t < nt; t++) th.emplace_back(work);
  } catch (...) {  // no more threads (or no memory for the list): the ones that exist, and this one, do the work
  }
  work();
  for (auto& t : th) t.join();
  return failed.load() == 0;
}

}  // namespace

extern "C" {

int ams_version(void) { return 200; }

const char* ams_strerror(int code) {
  switch (code) {
    case AMS_OK: return "ok";
    case AMS_ERR_FORMAT: return "unknown format";
    case AMS_ERR_SHAPE: return "shape or argument out of range";
    case AMS_ERR_NULL: return "null pointer";
    case AMS_ERR_ALIGN: return "device pointer not 16-byte aligned";
    case AMS_ERR_NONFINITE: return "weight is inf or NaN";
    case AMS_ERR_LAUNCH: return "kernel launch failed";
    case AMS_ERR_DEVICE: return "current device is not gfx950";
    case AMS_ERR_SCRATCH: return "problem too large for the library's static scratch (use ams_linear or ams_linear_ws)";
    case AMS_ERR_NOMEM: return "out of host memory";
    default: return "unknown error";
  }
}

int ams_group_size(int fmt) {
  const FormatInfo* fi = ams::format_info(fmt);
  return fi ? fi->group : 0;
}

int ams_code_bits(int fmt) {
  const FormatInfo* fi = ams::format_info(fmt);
  return fi ? fi->code_bits : 0;
}

int ams_packed_bytes(int fmt, int64_t N, int64_t K, size_t* bytes) {
  if (int rc = check_shape(fmt, N, K)) return rc;
  if (!bytes) return AMS_ERR_NULL;
  const FormatInfo& fi = *ams::format_info(fmt);
  *bytes = (size_t)ams::packed_bytes(fi, N, K);
  return AMS_OK;
}

int ams_canonical_bytes(int fmt, int64_t N, int64_t K, size_t* bytes) {
  if (int rc = check_shape(fmt, N, K)) return rc;
  if (!bytes) return AMS_ERR_NULL;
  switch (fmt) {
    case AMS_FMT_FP533_E2M3: *bytes = (size_t)2 * (size_t)((K + 2) / 3) * (size_t)N; break;     // one uint16 per 3 weights
    case AMS_FMT_FP425_E2M2: *bytes = (size_t)34 * (size_t)((K + 63) / 64) * (size_t)N; break;  // 17 uint16 per 64 weights
    case AMS_FMT_FP45_E2M2: *bytes = (size_t)9 * (size_t)((K + 15) / 16) * (size_t)N; break;    // 16 nibbles + 8 shared bits
    case AMS_FMT_FP433_E2M2: *bytes = (size_t)13 * (size_t)((K + 23) / 24) * (size_t)N; break;  // 24 nibbles + 8 shared bits
    case AMS_FMT_FP6_E2M3: *bytes = (size_t)3 * (size_t)((K + 3) / 4) * (size_t)N; break;       // 4 codes of 6 bits
    case AMS_FMT_FP5_E2M2: *bytes = (size_t)5 * (size_t)((K + 7) / 8) * (size_t)N; break;       // 8 codes of 5 bits
    default: *bytes = (size_t)((K + 1) / 2) * (size_t)N; break;                                 // FP4: 2 codes per byte
  }
  return AMS_OK;
}

int ams_pack(int fmt, const uint16_t* W, int64_t N, int64_t K, int64_t ldw, void* packed, uint16_t* scales,
             uint8_t* codes_out) {
  return ams_pack_ex(fmt, AMS_SEARCH_SET_BIT, W, N, K, ldw, packed, scales, codes_out);
}

namespace {
int pack_rows(int lanes, int fmt, int search, bool per_tensor, const uint16_t* W, int64_t N, int64_t K, int64_t ldw, void* packed,
              uint16_t* scales, uint8_t* codes_out);
}

int ams_pack_ex(int fmt, int search, const uint16_t* W, int64_t N, int64_t K, int64_t ldw, void* packed, uint16_t* scales,
                uint8_t* codes_out) {
  return pack_rows(kWidest, fmt, search, false, W, N, K, ldw, packed, scales, codes_out);
}

int ams_pack_per_tensor(int fmt, int search, const uint16_t* W, int64_t N, int64_t K, int64_t ldw, void* packed,
                        uint16_t* scales, uint8_t* codes_out) {
  return pack_rows(kWidest, fmt, search, true, W, N, K, ldw, packed, scales, codes_out);
}

namespace {
int pack_rows(int lanes, int fmt, int search, bool per_tensor, const uint16_t* W, int64_t N, int64_t K, int64_t ldw, void* packed,
              uint16_t* scales, uint8_t* codes_out) {
  if (int rc = check_shape(fmt, N, K)) return rc;
  if (search != AMS_SEARCH_SET_BIT && search != AMS_SEARCH_REROUND) return AMS_ERR_SHAPE;
  if (!W || !packed || !scales) return AMS_ERR_NULL;
  if (ldw < K) return AMS_ERR_SHAPE;
  const FormatInfo& fi = *ams::format_info(fmt);
  const RowQuant rq = {fmt, fi.code_bits - 3, fi.group, fi.fmax, search, wide_row(lanes)};
  const int64_t n_strips = ams::round_up(N, ams::kStripRows) / ams::kStripRows;
  uint16_t tensor_scale = 0;
  if (per_tensor) {  // Eq. 1 with the maximum over the whole matrix
    uint16_t absmax = 0;
    for (int64_t n = 0; n < N; n++) absmax = std::max(absmax, abs_max_bits(W + n * ldw, K));
    if (absmax >= 0x7C00) return AMS_ERR_NONFINITE;
    tensor_scale = scale_bits(absmax, fi.fmax);
  }
  std::atomic<int> bad{0};
  const WideRow* const wide = one_pass(rq, fi, K, codes_out);
  const bool done = parallel_for(n_strips, quantize_ns(rq, wide, N, K, K), [=, &fi, &bad](int64_t t) {
    Steps steps;
    if (wide) {
      if (!quantize_and_pack_strip(rq, fi, *wide, W, N, K, ldw, K, tensor_scale, (uint8_t*)packed, n_strips, t, steps,
                                   [&](int r, int64_t) { return scales + t * 16 + r; }))
        bad.store(1);
      return;
    }
    std::vector<uint8_t> buf((size_t)ams::kStripRows * K);
    const uint8_t* rows[16];
    for (int r = 0; r < 16; r++) {
      const int64_t n = t * 16 + r;
      if (n >= N) {
        rows[r] = nullptr;
        continue;
      }
      uint8_t* c = buf.data() + (size_t)r * K;
      if (!quantize_row(rq, W + n * ldw, K, c, scales + n, steps, tensor_scale)) bad.store(1);
      rows[r] = c;
      if (codes_out) std::memcpy(codes_out + n * K, c, (size_t)K);
    }
    pack_strip(fmt, rows, K, (uint8_t*)packed, n_strips, t);
  });
  if (!done) return AMS_ERR_NOMEM;
  return bad.load() ? AMS_ERR_NONFINITE : AMS_OK;
}
}  // namespace

// log2(scale_group / rec_k), or -1 when scale_group is not rec_k * 2^j
int scale_group_shift(const FormatInfo& fi, int64_t scale_group) {
  for (int j = 0; j < 20; j++)
    if (scale_group == (int64_t)fi.rec_k << j) return j;
  return -1;
}

int ams_group_scales_count(int fmt, int64_t N, int64_t K, int64_t scale_group, size_t* count) {
  if (int rc = check_shape(fmt, N, K)) return rc;
  if (!count) return AMS_ERR_NULL;
  const FormatInfo& fi = *ams::format_info(fmt);
  if (scale_group_shift(fi, scale_group) < 0) return AMS_ERR_SHAPE;
  *count = (size_t)(ams::round_up(N, ams::kStripRows)) * (size_t)((K + scale_group - 1) / scale_group);
  return AMS_OK;
}

namespace {
int pack_runs(int lanes, int fmt, int search, int64_t scale_group, const uint16_t* W, int64_t N, int64_t K, int64_t ldw,
              void* packed, uint16_t* scales, uint8_t* codes_out) {
  if (int rc = check_shape(fmt, N, K)) return rc;
  if (search != AMS_SEARCH_SET_BIT && search != AMS_SEARCH_REROUND) return AMS_ERR_SHAPE;
  if (!W || !packed || !scales) return AMS_ERR_NULL;
  if (ldw < K) return AMS_ERR_SHAPE;
  const FormatInfo& fi = *ams::format_info(fmt);
  if (scale_group_shift(fi, scale_group) < 0) return AMS_ERR_SHAPE;
  const RowQuant rq = {fmt, fi.code_bits - 3, fi.group, fi.fmax, search, wide_row(lanes)};
  const int64_t n_strips = ams::round_up(N, ams::kStripRows) / ams::kStripRows;
  const int64_t n_sg = (K + scale_group - 1) / scale_group;
  std::atomic<int> bad{0};
  const WideRow* const wide = one_pass(rq, fi, K, codes_out);
  const bool done = parallel_for(n_strips, quantize_ns(rq, wide, N, K, scale_group), [=, &fi, &bad](int64_t t) {
    Steps steps;
    if (wide) {
      auto scale_of = [&](int r, int64_t j) { return scales + ((size_t)t * n_sg + j) * 16 + r; };
      for (int r = 0; r < 16; r++)
        for (int64_t j = 0; j < n_sg && t * 16 + r >= N; j++) *scale_of(r, j) = 0x3C00;  // padding rows: 1.0
      if (!quantize_and_pack_strip(rq, fi, *wide, W, N, K, ldw, scale_group, 0, (uint8_t*)packed, n_strips, t, steps, scale_of)) bad.store(1);
      return;
    }
    std::vector<uint8_t> buf((size_t)ams::kStripRows * K);
    const uint8_t* rows[16];
    for (int r = 0; r < 16; r++) {
      const int64_t n = t * 16 + r;
      uint16_t* srow = scales + (size_t)t * n_sg * 16 + r;  // [strip][run][row in strip]
      if (n >= N) {
        rows[r] = nullptr;
        for (int64_t j = 0; j < n_sg; j++) srow[j * 16] = 0x3C00;  // padding rows: 1.0
        continue;
      }
      uint8_t* c = buf.data() + (size_t)r * K;
      for (int64_t j = 0; j < n_sg; j++) {  // Eq. 1 and the search on every run by itself
        const int64_t a = j * scale_group, len = std::min<int64_t>(scale_group, K - a);
        if (!quantize_row(rq, W + n * ldw + a, len, c + a, srow + j * 16, steps)) bad.store(1);
      }
      rows[r] = c;
      if (codes_out) std::memcpy(codes_out + n * K, c, (size_t)K);
    }
    pack_strip(fmt, rows, K, (uint8_t*)packed, n_strips, t);
  });
  if (!done) return AMS_ERR_NOMEM;
  return bad.load() ? AMS_ERR_NONFINITE : AMS_OK;
}

}  // namespace

int ams_pack_grouped(int fmt, int search, int64_t scale_group, const uint16_t* W, int64_t N, int64_t K, int64_t ldw,
                     void* packed, uint16_t* scales, uint8_t* codes_out) {
  return pack_runs(kWidest, fmt, search, scale_group, W, N, K, ldw, packed, scales, codes_out);
}

// Not in the header, for the tests: the packer as a processor with vectors of at most `lanes` groups (16, 8 or 0) runs it.
// scale_group: weights per scale, 0: a scale per row, -1: one for the matrix.  AMS_ERR_DEVICE: this processor's vectors
// are shorter.
int ams_pack_lanes(int lanes, int fmt, int search, int64_t scale_group, const uint16_t* W, int64_t N, int64_t K, int64_t ldw,
                   void* packed, uint16_t* scales, uint8_t* codes_out) {
  const WideRow* const vectors = wide_row(lanes);
  if (lanes != (vectors ? vectors->lanes : 0)) return AMS_ERR_DEVICE;
  if (scale_group > 0) return pack_runs(lanes, fmt, search, scale_group, W, N, K, ldw, packed, scales, codes_out);
  return pack_rows(lanes, fmt, search, scale_group < 0, W, N, K, ldw, packed, scales, codes_out);
}

int ams_pack_codes(int fmt, const uint8_t* codes, int64_t N, int64_t K, void* packed) {
  if (int rc = check_shape(fmt, N, K)) return rc;
  if (!codes || !packed) return AMS_ERR_NULL;
  const FormatInfo& fi = *ams::format_info(fmt);
  const int64_t n_strips = ams::round_up(N, ams::kStripRows) / ams::kStripRows;
  std::atomic<int> bad{0};
  parallel_for(n_strips, (double)N * K * kPackCodesNs, [=, &fi, &bad](int64_t t) {
    const uint8_t* rows[16];
    for (int r = 0; r < 16; r++) {
      const int64_t n = t * 16 + r;
      rows[r] = n < N ? codes + n * K : nullptr;
      if (n >= N) continue;
      for (int64_t k0 = 0; k0 < K; k0 += fi.group) {
        const int64_t k1 = std::min<int64_t>(K, k0 + fi.group);
        for (int64_t k = k0; k < k1; k++)
          if ((rows[r][k] >> fi.code_bits) || ((rows[r][k] ^ rows[r][k0]) & 1)) bad.store(1);
      }
    }
    pack_strip(fmt, rows, K, (uint8_t*)packed, n_strips, t);
  });
  return bad.load() ? AMS_ERR_SHAPE : AMS_OK;
}

int ams_unpack_host(int fmt, const void* packed, int64_t N, int64_t K, uint8_t* codes) {
  if (int rc = check_shape(fmt, N, K)) return rc;
  if (!codes || !packed) return AMS_ERR_NULL;
  const FormatInfo& fi = *ams::format_info(fmt);
  const int64_t n_strips = ams::round_up(N, ams::kStripRows) / ams::kStripRows;
  parallel_for(n_strips, (double)N * K * kUnpackNs, [=, &fi](int64_t t) {
    uint8_t* rows[16];
    for (int r = 0; r < 16; r++) rows[r] = t * 16 + r < N ? codes + (t * 16 + r) * K : nullptr;
    unpack_strip(fmt, fi, (const uint8_t*)packed, n_strips, t, K, rows);
  });
  return AMS_OK;
}

}  // extern "C"
