// HIP kernels (gfx950 / CDNA4) of the AMS-Quant weight-only quantized Linear:
// bit-level restoration of the packed weights (Sec. 3.2, Sec. 3.3 stages 2-3) fused
// with the skinny fp16 matmul of the decode stage (Sec. 4.2), and the fp16 baseline.
//
// Every lane loads its 16-byte chunk of a record with one dwordx4 (a record is one
// contiguous 1 KiB access per wavefront), restores the fp16 pairs in registers and feeds
// them as the A operand of v_mfma_f32_16x16x32_f16; the activations are staged in LDS in
// the operand order the restoration produces.
//   slice_kernel   (ams_slice.hip) the packed formats, most shapes: wavefronts share K, activations
//                  streamed beside the weights.
//   column_kernel  the packed formats otherwise: a workgroup owns up to 16 neighbouring strips, every
//                  wavefront stays with one strip and walks K in step with all the others, so
//                  that the grid as a whole reads one contiguous, moving window of the K-major
//                  packed matrix; the partial tile of a strip never leaves its wavefront's
//                  registers until the end.
//   sweep_kernel / stream_kernel   the fp16 baseline (row-major weights).
// Partial tiles are combined through LDS, deterministically; only the entry points that take
// a workspace also split K over workgroups and exchange fp32 tiles through it.
#include <algorithm>
#include <type_traits>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <unordered_set>

#include "ams_device.h"

namespace {
using namespace ams_dev;

// Activation staging.  A wave copies X[0..M) x [k0, k0+nk) into its LDS region in operand
// order (zero beyond K), nk a multiple of the record size.  The copy is split in a load
// half (global -> registers, no control flow around the loads) and a store half
// (permute + LDS write) so that the loads can be issued ahead of the weight stream.
// The work is cut in units of UNIT halfs; unit u covers row u >> x_shift, position
// u & (2^x_shift - 1) (rows are padded to a power of two of units).
template <int FMT>
struct XUnit {
  static constexpr int UNIT = Fmt<FMT>::PB;               // halfs permuted together
  static constexpr int CH = UNIT / 8;                     // 16-byte chunks per unit
  static constexpr int XU = 2;                            // units a lane moves in the first pass (in flight with the weights)
  static constexpr int XB = CH == 1 ? 8 : CH == 2 ? 4 : 2;  // units a lane moves in each further pass (all requested, then stored)
};

template <int FMT, int NU = XUnit<FMT>::XU>
struct XRegs {
  u4 c[NU][XUnit<FMT>::CH];
};

// Units u0 + i * nthr + idx, i < NU.
// RAGGED: rows of X start anywhere (K no multiple of 8, at least 8); a chunk that runs past its row's end is read from
// the row's last eight channels and shifted into place by x_store.  11003 x 4099 at M = 5: 9.7 us; 23.5 us when such
// rows went element by element (a division and a search for its slot each).
template <bool RAGGED = false, int FMT, int NU>
__device__ __forceinline__ void x_load(XRegs<FMT, NU>& xr, const LinearArgs& a, int k0, int nk, int u0, int idx, int nthr) {
  constexpr int UNIT = XUnit<FMT>::UNIT, CH = XUnit<FMT>::CH;
  const int upr = nk / UNIT;
#pragma unroll
  for (int i = 0; i < NU; i++) {
    const int u = u0 + i * nthr + idx;
    const int m = u >> a.x_shift, j = u & ((1 << a.x_shift) - 1);
    const int k = k0 + UNIT * j;
    const bool row_ok = m < a.M && j < upr;
#pragma unroll
    for (int e = 0; e < CH; e++) {
      const bool ok = row_ok && k + 8 * e < a.K;
      // redirected loads are zeroed by x_store
      if constexpr (RAGGED) {
        const size_t off = ok ? (size_t)m * a.K + min(k + 8 * e, a.K - 8) : 0;
        __builtin_memcpy(&xr.c[i][e], a.X + off, 16);  // one unaligned load
      } else {
        const size_t off = ok ? (size_t)m * a.K + k + 8 * e : 0;
        xr.c[i][e] = *(const u4*)(a.X + off);
      }
    }
  }
}

template <bool RAGGED = false, int FMT, int NU>
__device__ __forceinline__ void x_store(const XRegs<FMT, NU>& xr, _Float16* xs, const LinearArgs& a, int k0, int nk, int u0,
                                        int idx, int nthr) {
  constexpr int UNIT = XUnit<FMT>::UNIT, CH = XUnit<FMT>::CH;
  const int upr = nk / UNIT;
#pragma unroll
  for (int i = 0; i < NU; i++) {
    const int u = u0 + i * nthr + idx;
    const int m = u >> a.x_shift, j = u & ((1 << a.x_shift) - 1);
    const int k = k0 + UNIT * j;
    uint32_t in[4 * CH], out[4 * CH];
#pragma unroll
    for (int e = 0; e < CH; e++) {
      const uint32_t keep = k + 8 * e < a.K ? 0xFFFFFFFFu : 0u;  // zero beyond K
      in[4 * e] = xr.c[i][e][0] & keep, in[4 * e + 1] = xr.c[i][e][1] & keep;
      in[4 * e + 2] = xr.c[i][e][2] & keep, in[4 * e + 3] = xr.c[i][e][3] & keep;
      if constexpr (RAGGED) shift_tail(&in[4 * e], k + 8 * e + 8 - a.K);
    }
    permute_unit<FMT>(in, out);
    if (m < a.M && j < upr) {
      u4* dst = (u4*)(xs + m * a.x_stride + UNIT * j);
#pragma unroll
      for (int e = 0; e < CH; e++) dst[e] = u4{out[4 * e], out[4 * e + 1], out[4 * e + 2], out[4 * e + 3]};
    }
  }
}

// Element-by-element staging for rows shorter than one 16-byte load (K < 8).
template <int FMT>
__device__ __forceinline__ void stage_x_short(_Float16* xs, const LinearArgs& a, int k0, int nk, int idx0, int nthr) {
  for (int idx = idx0; idx < a.M * nk; idx += nthr) {
    const int m = idx / nk, kk = idx - m * nk;
    const int k = k0 + kk;
    const uint16_t v = k < a.K ? a.X[(size_t)m * a.K + k] : (uint16_t)0;
    const int rl = kk / Fmt<FMT>::REC_K, kr = kk - rl * Fmt<FMT>::REC_K;
    ((uint16_t*)xs)[m * a.x_stride + rl * Fmt<FMT>::REC_K + x_slot<FMT>(kr)] = v;
  }
}

// fp16 bits of the scales of the four output channels a lane holds of a strip's tile
struct ScaleBits {
  uint16_t b[4];
};
template <int FMT>
__device__ __forceinline__ ScaleBits load_scale_bits(const LinearArgs& a, int strip, int lane) {
  ScaleBits sb = {{0x3C00, 0x3C00, 0x3C00, 0x3C00}};
  if constexpr (FMT != FMT_FP16) {
    const int n0 = strip * 16 + 4 * (lane >> 4);
#pragma unroll
    for (int r = 0; r < 4; r++) sb.b[r] = a.scales[min(n0 + r, a.N - 1)];  // clamped: rows beyond N are never stored
  }
  return sb;
}
// fp32 multipliers s_n * 2^14 (the baseline's "scales" are 1: its bits are 1.0 and no 2^14 is owed)
__device__ __forceinline__ f4 scales_from_bits(const ScaleBits& sb, float mul = kTwo14) {
  f4 sc;
#pragma unroll
  for (int r = 0; r < 4; r++) sc[r] = (float)__builtin_bit_cast(_Float16, sb.b[r]) * mul;
  return sc;
}
template <int FMT>
__device__ __forceinline__ f4 load_scales(const LinearArgs& a, int strip, int lane) {
  return scales_from_bits(load_scale_bits<FMT>(a, strip, lane), FMT == FMT_FP16 ? 1.0f : kTwo14);
}

// Multiply a finished 16x16 tile (C[i][j]: lane = j + 16*(i/4), register i%4) by the scales, convert, store.
template <int MT>
__device__ __forceinline__ void store_tile_scaled(const f4 t[MT], const f4 sc, const LinearArgs& a, int strip, int lane) {
  const int m_lo = lane & 15, kq = lane >> 4;
#pragma unroll
  for (int mt = 0; mt < MT; mt++) {
    const int m = m_lo + 16 * mt;
    if (m < a.M) {
      const int n0 = strip * 16 + 4 * kq;
      us4 h;
#pragma unroll
      for (int r = 0; r < 4; r++) h[r] = __builtin_bit_cast(uint16_t, (_Float16)(t[mt][r] * sc[r]));
      if (n0 + 3 < a.N && (a.N & 3) == 0) {  // the lane's four output channels are eight aligned bytes of Y's row m
        *(us4*)(a.Y + (size_t)m * a.N + n0) = h;
      } else {
#pragma unroll
        for (int r = 0; r < 4; r++)
          if (n0 + r < a.N) a.Y[(size_t)m * a.N + n0 + r] = h[r];
      }
    }
  }
}

// K is split over gk workgroups: every one leaves its partial tile in the workspace and counts itself in; the one that
// arrives last adds all gk tiles in slice order (so the result does not depend on who was last) and clears the counter
// for the next call.  Nobody waits for anybody.  True, with the sum, for the one that arrived last.
// The tiles travel by stores and loads with the device's cache policy (they go to the level of the memory system all
// compute units share).  What orders them: the wave waits until every one of its tile stores has been acknowledged
// (s_waitcnt vmcnt(0): on this target stores count in vmcnt) before it counts itself in, and the last arriver's tile loads
// are issued only after its own count has come back (the branch below depends on it).  A device-scope fence would
// instead write back and invalidate the whole L2, which costs more than the Linear itself.
// 16 bytes per lane, and the tiles of all slices are asked for before the first is added: element by element and slice by
// slice every one of them was a trip to memory (7168 x 8192 FP5.33 M = 16, four slices, 14.4 -> 12.8 us).
template <int MT>
__device__ __forceinline__ bool exchange_tile(const LinearArgs& a, int gk, int strip, f4 (&sum)[MT], int lane) {
  const __amdgpu_buffer_rsrc_t tiles = __builtin_amdgcn_make_buffer_rsrc((void*)a.ws_tiles, 0, a.gk * a.n_strips * MT * 1024, 0x00020000);
  auto offset = [&](int slice, int t) { return (((slice * a.n_strips + strip) * MT + t) * 64 + lane) * 16; };
#pragma unroll
  for (int t = 0; t < MT; t++) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, sum[t]), tiles, offset(gk, t), 0, kDeviceScope);
  // all tile stores of this wave acknowledged; the compiler moves no memory access across either statement
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  unsigned before = 0;
  if (lane == 0) before = __hip_atomic_fetch_add(a.ws_count + strip, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  before = __builtin_amdgcn_readfirstlane(before);
  if (before != (unsigned)a.gk - 1) return false;
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the count has returned; the tile loads below are issued after it
  // With two row tiles four slices are in registers at a time, the second four only where they exist:
  // all eight would be 64 registers, which workgroups of 1024 threads have only with spills (10 column
  // kernels spilled, now 5).  8192 x 14337 FP6 M = 32 in four slices 33.1 -> 32.6 us, 5120 x 10008 FP4.33
  // M = 24 15.1 -> 14.9; with eight slices one trip more, 1000 x 14337 FP5.33 M = 24 12.7 -> 12.9.
  constexpr int AT_ONCE = kMaxSlices / MT;
#pragma unroll
  for (int t = 0; t < MT; t++) sum[t] = f4{0, 0, 0, 0};
#pragma unroll
  for (int q0 = 0; q0 < kMaxSlices; q0 += AT_ONCE) {
    if (q0 > 0 && q0 >= a.gk) break;
    f4 part[AT_ONCE][MT];
#pragma unroll
    for (int q = 0; q < AT_ONCE; q++)
#pragma unroll
      for (int t = 0; t < MT; t++)  // slices that do not exist read nothing and add 0
        part[q][t] = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(tiles, q0 + q < a.gk ? offset(q0 + q, t) : kOutOfRange, 0, kDeviceScope));
#pragma unroll
    for (int t = 0; t < MT; t++)
#pragma unroll
      for (int q = 0; q < AT_ONCE; q++) sum[t] += part[q][t];
  }
  if (lane == 0) __hip_atomic_store(a.ws_count + strip, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return true;
}

// The streaming Linear.  A workgroup owns `spw` consecutive strips and walks K in
// phases of `rc` records per strip (one phase when the activations M x K fit in LDS).
// Inside a phase its work is the list of (strip, record) pairs in strip-major order;
// the S wavefronts cut that list into S equal contiguous pieces, whatever the strip
// boundaries, so every wave streams the same number of bytes through its register ring
// (records of a strip are adjacent in memory, and with one phase those of consecutive
// strips are too).  The pieces are the same in every phase, so a wave meets the same
// strips again: its partial 16x16 tiles live in LDS slots and are swapped in and out
// of the accumulator registers where its piece crosses a strip boundary.  The
// activations of a phase are staged once per workgroup in LDS (operand order).  After
// the last phase the wave holding a strip's first record adds the tiles of the waves
// after it, in wave order, scales and stores.  The grid is one resident round.
template <int MT, int LR>
__global__ void __launch_bounds__(1024) stream_kernel(LinearArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int FMT = FMT_FP16;  // the baseline's kernel: row-major fp16 weights
  constexpr int REC_K = Fmt<FMT>::REC_K;
  // All kernel arguments are pulled in at once: fetched piecemeal where they are first used,
  // each batch would be one more trip to memory in front of the first weight load.
  asm volatile("" ::"s"(a.W), "s"(a.scales), "s"(a.X), "s"(a.Y), "s"(a.M), "s"(a.N), "s"(a.K), "s"(a.n_rec), "s"(a.x_stride),
               "s"(a.x_region), "s"(a.x_shift), "s"(a.n_strips), "s"(a.spw), "s"(a.red_slots), "s"(a.piece_q), "s"(a.piece_r),
               "s"(a.rc));
  const int tid = threadIdx.x, lane = tid & 63, nthr = blockDim.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int S = nthr >> 6;
  const int strip0 = blockIdx.x * a.spw;
  const int ns = min(a.spw, a.n_strips - strip0);
  const int RC = a.rc;
  const int P = ns * RC;  // (strip, record) pairs of one phase
  // balanced pieces: wave w takes piece_q pairs, the first piece_r waves one more
  // (the host supplies the quotient for full workgroups: no 64-bit division in here)
  int piece_q = a.piece_q, piece_r = a.piece_r;
  if (ns != a.spw) {
    piece_q = (int)((unsigned)P / (unsigned)S);
    piece_r = P - piece_q * S;
  }
  const int g0 = wave * piece_q + min(wave, piece_r), g1 = g0 + piece_q + (wave < piece_r ? 1 : 0);
  const int g_last = max(g1 - 1, 0);
  // strip of the piece's first pair and its record inside the phase
  const int s_first = (int)((unsigned)min(g0, g_last) / (unsigned)RC);
  const int j_first = min(g0, g_last) - s_first * RC;
  _Float16* xs = (_Float16*)smem;
  f4* red = (f4*)(smem + (size_t)a.x_region * 2);  // [S][red_slots][MT][64]
  f4* const my_red = red + (size_t)wave * a.red_slots * MT * 64 + lane;  // this wave's tiles: [slot][MT][64]
  const int m_lo = lane & 15, kq = lane >> 4;
  const int lane_off = FMT == FMT_FP16 ? 8 * kq : (REC_K / 4) * kq;
  // lanes whose activation row does not exist read row 0: they only feed output columns never stored
  const _Float16* x0 = xs + (m_lo < a.M ? m_lo : 0) * a.x_stride + lane_off;
  const _Float16* x1 = xs + (m_lo + 16 < a.M ? m_lo + 16 : 0) * a.x_stride + lane_off;

  const int total_units = a.M << a.x_shift;
  const int units_per_pass = nthr * XUnit<FMT>::XU;
  const bool wave_has_x = wave * 64 < total_units;  // wave-uniform
  const int chunk_k = RC * REC_K;
  __builtin_amdgcn_sched_barrier(0);

  for (int rec_base = 0; rec_base < a.n_rec; rec_base += RC) {
    // Activations of the phase, in operand order.  Units beyond the first pass (large M)
    // are staged by a loop that runs to completion first; the first pass is only requested here and stored after the head of the weight stream has
    // been requested too, so both are in flight together and the stream starts as soon
    // as its first record lands.  Waves whose units all fall outside skip the pass.
    if (rec_base > 0) __syncthreads();  // everyone is done with the previous phase's activations
    const int k0 = rec_base * REC_K;
    XRegs<FMT> xr;
    for (int u0 = units_per_pass; u0 < total_units; u0 += nthr * XUnit<FMT>::XB) {
      XRegs<FMT, XUnit<FMT>::XB> xb;
      x_load(xb, a, k0, chunk_k, u0, tid, nthr);
      x_store(xb, xs, a, k0, chunk_k, u0, tid, nthr);
    }
    if (wave_has_x) x_load(xr, a, k0, chunk_k, 0, tid, nthr);
    __builtin_amdgcn_sched_barrier(0);

    // the head of the weight stream: LR records in flight per wave.  The prefetch cursor
    // (pair index, strip, record in phase) is clamped to the piece's last pair; records
    // beyond the end of K (last phase) are redirected to the strip's last record and skipped.
    const int rec_hi = a.n_rec - 1 - rec_base;  // last valid record of this phase, relative
    int pp = min(g0, g_last), ps = s_first, pj = j_first;
    LaneRec<FMT> ring[LR];
#pragma unroll
    for (int q = 0; q < LR; q++) {
      load_rec<FMT>(ring[q], a, strip0 + ps, rec_base + min(pj, rec_hi), lane);
      if (pp < g_last) {
        pp++;
        if (++pj == RC) pj = 0, ps++;
      }
      __builtin_amdgcn_sched_barrier(0);  // issue in ring order: the oldest load is the first one needed
    }

    if (rec_base == 0) {
      // set-up that nothing above needs, done while the first loads are in flight: this wave's tile slots cleared
      for (int t = 0; t < a.red_slots * MT; t++) my_red[t * 64] = f4{0, 0, 0, 0};
    }
    if (wave_has_x) x_store(xr, xs, a, k0, chunk_k, 0, tid, nthr);
    __syncthreads();

    f4 acc[MT];
    f4* slot_ptr = my_red;
#pragma unroll
    for (int i = 0; i < MT; i++) acc[i] = slot_ptr[i * 64];
    int g = g0, j = j_first;

    // One pair: multiply, refill the ring slot; where the strip (or the piece) ends, the
    // tile goes back to its LDS slot and the next strip's tile comes in.  Nothing in
    // here touches global memory except the refill, so the ring drains one record at a time.
    auto step = [&](LaneRec<FMT>& slot) {
      if (j <= rec_hi) mac_rec<FMT, MT>(slot, x0 + j * REC_K, x1 + j * REC_K, acc);
      load_rec<FMT>(slot, a, strip0 + ps, rec_base + min(pj, rec_hi), lane);
      if (pp < g_last) {
        pp++;
        if (++pj == RC) pj = 0, ps++;
      }
      g++;
      j++;
      if (j == RC || g == g1) {
#pragma unroll
        for (int i = 0; i < MT; i++) slot_ptr[i * 64] = acc[i];
        if (j == RC) {
          slot_ptr += MT * 64;
          j = 0;
        }
#pragma unroll
        for (int i = 0; i < MT; i++) acc[i] = slot_ptr[i * 64];
      }
    };

    while (g + LR <= g1) {
#pragma unroll
      for (int q = 0; q < LR; q++) {
        step(ring[q]);
        // keep the refill right behind its record
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int q = 0; q < LR - 1; q++)
      if (g < g1) step(ring[q]);
  }

  // Finish the strips.  The wave that holds a strip's first pair owns it: it adds the
  // head tiles (slot 0) of the waves after it whose pieces still lie in that strip, in
  // wave order, and stores.  The tile reads do not depend on each other, so they overlap.
  __syncthreads();
  if (g1 > g0) {
    const int s_begin = j_first == 0 ? s_first : s_first + 1;  // first strip that starts inside this piece
    for (int s = s_begin; s * RC < g1; s++) {
      const int se = (s + 1) * RC;
      f4 sum[MT];
#pragma unroll
      for (int i = 0; i < MT; i++) sum[i] = red[(((size_t)wave * a.red_slots + (s - s_first)) * MT + i) * 64 + lane];
      if (se > g1) {  // the strip runs on into the pieces of the next nf waves
        int nf = 0;
        for (int w2 = wave + 1, h0 = g1; w2 < S && h0 < se; w2++) {
          const int len = piece_q + (w2 < piece_r ? 1 : 0);
          if (len == 0) break;
          h0 += len;
          nf++;
        }
        const f4* follower = red + (size_t)wave * a.red_slots * MT * 64 + lane;  // slot 0 of this wave; followers are whole waves further
        const int wave_stride = a.red_slots * MT * 64;
#pragma unroll
        for (int d = 1; d < 16; d++) {
          // reads are independent and unconditional (inside the tile area: wave index clamped);
          // selected, not multiplied: a tile that is not taken may be uninitialised LDS
          const f4* t = follower + min(d, S - 1 - wave) * wave_stride;
#pragma unroll
          for (int i = 0; i < MT; i++) {
            const f4 v = t[i * 64];
            sum[i] += d <= nf ? v : f4{0, 0, 0, 0};
          }
        }
      }
      store_tile_scaled<MT>(sum, f4{1.0f, 1.0f, 1.0f, 1.0f}, a, strip0 + s, lane);  // the baseline has no scales
    }
  }
}

// The sweeping Linear.  Strips are dealt to the workgroups round robin (workgroup g owns
// strips g, g + G, g + 2G, ...), and inside a workgroup the records of its strips, taken
// as one list in that order, are dealt to the S wavefronts record by record.  At any
// moment a workgroup therefore reads one contiguous run of S * LR records, and the whole
// grid reads a window of G neighbouring strips that moves through the matrix front to
// back: the order the memory system serves fastest (measured with bare read kernels, this
// beats per-wavefront contiguous pieces by 15-20 % on the Llama shapes, and two records in
// flight per wave beat four).  Every wave meets every strip of its workgroup, so it parks
// one partial 16x16 tile per strip in LDS (only the lanes of existing activation rows);
// after one barrier the strips are finished one per wave: the S tiles added in wave
// order, scaled, converted, stored.  The activations are staged once per workgroup in LDS
// in operand order; when M x K does not fit, K is walked in phases of rc records per strip
// and the parked tiles accumulate over the phases.  The grid is one resident round.
template <int MT, int LR, bool GROUPS = false>
__global__ void __launch_bounds__(1024) sweep_kernel(LinearArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int FMT = FMT_FP16;  // the baseline's kernel: row-major fp16 weights
  constexpr int REC_K = Fmt<FMT>::REC_K;
  asm volatile("" ::"s"(a.W), "s"(a.scales), "s"(a.X), "s"(a.Y), "s"(a.M), "s"(a.N), "s"(a.K), "s"(a.n_rec), "s"(a.x_stride),
               "s"(a.x_region), "s"(a.x_shift), "s"(a.n_strips), "s"(a.spw), "s"(a.rc), "s"(a.gn), "s"(a.gk), "s"(a.wps));
  const int tid = threadIdx.x, lane = tid & 63, nthr = blockDim.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int S = nthr >> 6;
  // workgroup = (position g along N, slice gk of K); without a split the grid is all along N
  const int G = a.gn;
  const int gk = a.gk > 1 ? (int)(blockIdx.x / (unsigned)G) : 0;
  const int g = (int)blockIdx.x - gk * G;
  const int ns = (a.n_strips - g + G - 1) / G;  // strips of this workgroup (>= 1)
  const int RC = a.rc;                          // records per strip in one phase of K
  // records [rec_lo, rec_hi) of every strip are this workgroup's slice of K
  const int rec_lo = a.gk > 1 ? (int)((unsigned)(gk * a.n_rec) / (unsigned)a.gk) : 0;
  const int rec_hi = a.gk > 1 ? (int)((unsigned)((gk + 1) * a.n_rec) / (unsigned)a.gk) : a.n_rec;
  const bool one_phase = RC >= rec_hi - rec_lo;
  const int mc = min(a.M, 16);  // activation rows of an MFMA tile that exist
  _Float16* xs = (_Float16*)smem;
  f4* parts = (f4*)(smem + (size_t)a.x_region * 2);  // [spw][wps][MT][4 K-quarters][mc]
  // The waves come in S / wps groups of wps; group vs owns the local strips vs, vs + sg, ...
  // and deals their records to its waves one by one (wps = S: all waves on one strip at a
  // time; fewer when the parked tiles, one per strip and wave of its group, must be fewer).
  // (GROUPS = false is the common case wps = S, spelled out so that it costs nothing.)
  const int wps = GROUPS ? a.wps : S;
  const int sg = GROUPS ? S / wps : 1;
  const int vs = GROUPS ? (int)((unsigned)wave / (unsigned)wps) : 0, vw = wave - vs * wps;
  const int ns_v = vs < ns ? (ns - vs + sg - 1) / sg : 0;  // strips of this wave's group
  // the group's j-th strip is local strip vs + j * sg = strip strip0 + j * strip_step of the
  // matrix; a group without strips reads (only reads) the workgroup's first strip
  const int strip0 = g + (ns_v > 0 ? vs : 0) * G, strip_step = (ns_v > 0 ? sg : 0) * G;
  const int m_lo = lane & 15, kq = lane >> 4;
  const int lane_off = FMT == FMT_FP16 ? 8 * kq : (REC_K / 4) * kq;
  // lanes whose activation row does not exist read row 0: they only feed output columns never stored
  const _Float16* x0 = xs + (m_lo < a.M ? m_lo : 0) * a.x_stride + lane_off;
  const _Float16* x1 = xs + (m_lo + 16 < a.M ? m_lo + 16 : 0) * a.x_stride + lane_off;
  const int part_f4 = MT * 4 * mc;  // f4 per parked tile
  // this wave's tile of its group's first strip; the next strips' tiles follow part_step apart
  f4* const my_part = parts + (size_t)((ns_v > 0 ? vs : 0) * wps + vw) * part_f4 + kq * mc + m_lo;
  const int part_step = sg * wps * part_f4;

  const int total_units = a.M << a.x_shift;
  const int units_per_pass = nthr * XUnit<FMT>::XU;
  const bool wave_has_x = wave * 64 < total_units;  // wave-uniform
  const int chunk_k = RC * REC_K;
  __builtin_amdgcn_sched_barrier(0);

  // K is walked in phases of RC records per strip (one phase when all activations fit in LDS).
  for (int rec_base = rec_lo; rec_base < rec_hi; rec_base += RC) {
    const int n_rec = min(RC, rec_hi - rec_base);                 // records per strip in this phase
    const int total = ns_v * n_rec;                                  // records of this wave's group
    const int cnt = vw < total ? (total - vw + wps - 1) / wps : 0;  // records of this wave
    if (rec_base > rec_lo) __syncthreads();  // everyone is done with the previous phase's activations
    const int k0 = rec_base * REC_K;

    // Activations: units beyond the first pass (large M) are staged by a loop that
    // runs to completion; the first pass is only requested here and stored behind the
    // head of the weight stream, so both are in flight together.
    XRegs<FMT> xr;
    for (int u0 = units_per_pass; u0 < total_units; u0 += nthr * XUnit<FMT>::XB) {
      XRegs<FMT, XUnit<FMT>::XB> xb;
      x_load(xb, a, k0, chunk_k, u0, tid, nthr);
      x_store(xb, xs, a, k0, chunk_k, u0, tid, nthr);
    }
    if (wave_has_x) x_load(xr, a, k0, chunk_k, 0, tid, nthr);
    __builtin_amdgcn_sched_barrier(0);

    // Head of the weight stream.  The prefetch cursor (position in the list, local strip,
    // record) stops at the wave's last record; a wave without records reads record 0.
    int pf = vw < total ? vw : 0, pj = 0, pr = pf;
    while (pr >= n_rec) pr -= n_rec, pj++;
    int cj = pj, cr = pr;  // strip (counted inside the group) and record (inside the phase) being multiplied

    // LR records are in flight while a record is being restored: the ring has one slot more,
    // and a step first requests the record LR places ahead into the slot freed by the step
    // before, then works on its own (a refill into the slot being read would have to wait
    // until the restoration has consumed it).
    constexpr int RS = LR + 1;
    struct Slot {
      LaneRec<FMT> r;
    };
    Slot ring[RS];
    auto request = [&](Slot& slot) {
      const int strip = strip0 + pj * strip_step;
      load_rec<FMT, false>(slot.r, a, strip, rec_base + pr, lane);
      if (pf + wps < total) {
        pf += wps, pr += wps;
        while (pr >= n_rec) pr -= n_rec, pj++;
      }
    };
#pragma unroll
    for (int q = 0; q < LR; q++) {
      request(ring[q]);
      __builtin_amdgcn_sched_barrier(0);  // issue in ring order: the oldest load is the first one needed
    }

    // while those are in flight: every tile slot cleared (a wave need not meet every strip when a
    // strip has fewer records than the workgroup has waves)
    if (rec_base == rec_lo)
      for (int i = tid; i < ns * wps * part_f4; i += nthr) parts[i] = f4{0, 0, 0, 0};
    if (wave_has_x) x_store(xr, xs, a, k0, chunk_k, 0, tid, nthr);
    __syncthreads();

    f4 acc[MT];
#pragma unroll
    for (int i = 0; i < MT; i++) acc[i] = f4{0, 0, 0, 0};
    bool pending = false;  // acc holds products that are not parked yet

    auto park = [&]() {
      if (m_lo < mc) {
        f4* t = my_part + cj * part_step;
        if (one_phase) {
#pragma unroll
          for (int i = 0; i < MT; i++) t[i * 4 * mc] = acc[i];
        } else {  // the slot belongs to this wave alone: a plain read-add-write
#pragma unroll
          for (int i = 0; i < MT; i++) t[i * 4 * mc] += acc[i];
        }
      }
#pragma unroll
      for (int i = 0; i < MT; i++) acc[i] = f4{0, 0, 0, 0};
    };
    // One record: request the one LR ahead, multiply, move on by S records; where that leaves
    // the strip, the tile is parked.  Only the request touches global memory.
    auto step = [&](Slot& slot, Slot& free_slot) {
      request(free_slot);
      __builtin_amdgcn_sched_barrier(0);
      mac_rec<FMT, MT>(slot.r, x0 + cr * REC_K, x1 + cr * REC_K, acc);
      pending = true;
      cr += wps;
      if (cr >= n_rec) {
        park();
        pending = false;
        do {
          cr -= n_rec, cj++;
        } while (cr >= n_rec);
      }
    };

    int i = 0;
    for (; i + RS <= cnt; i += RS) {
#pragma unroll
      for (int q = 0; q < RS; q++) {
        step(ring[q], ring[(q + LR) % RS]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int q = 0; q < RS - 1; q++)
      if (i + q < cnt) step(ring[q], ring[(q + LR) % RS]);
    if (pending) park();
  }

  // Finish the strips, one per wave: the wps parked tiles added in wave order.
  __syncthreads();
  for (int j = wave; j < ns; j += S) {
    f4 sum[MT];
#pragma unroll
    for (int t = 0; t < MT; t++) sum[t] = f4{0, 0, 0, 0};
    if (m_lo < mc) {
      const f4* t0 = parts + (size_t)j * wps * part_f4 + kq * mc + m_lo;
      for (int w = 0; w < wps; w++) {
#pragma unroll
        for (int t = 0; t < MT; t++) sum[t] += t0[(size_t)w * part_f4 + t * 4 * mc];
      }
    }
    const int strip = g + j * G;
    if (a.gk > 1 && !exchange_tile<MT>(a, gk, strip, sum, lane)) continue;
    store_tile_scaled<MT>(sum, f4{1.0f, 1.0f, 1.0f, 1.0f}, a, strip, lane);  // the baseline has no scales
  }
}

// The fp16 baseline at small batches (Sec. 4.2's W16A16 GEMV): every wavefront owns whole rows of the
// row-major matrix, dealt round robin over all wavefronts of the grid, and reads a row as consecutive
// 1 KiB segments (one 16-byte load per lane, LR of them in flight), multiplies on the VALU (packed dot
// products into fp32, the lane's eight channels against the same eight of each activation row in LDS)
// and adds the 64 lanes of a row up when the row ends.  a.x_stride = halfs between activation rows in
// LDS (K rounded up to whole segments; the tail is zero).  K is a multiple of 8.
template <int MB, bool NT>
__global__ void __launch_bounds__(1024) gemv_fp16_kernel(LinearArgs a) {
  extern __shared__ __align__(16) uint8_t smem[];
  typedef _Float16 h2 __attribute__((ext_vector_type(2)));
  constexpr int LR = 2, RS = LR + 1, SEG = 512;  // halfs of a row one wavefront load covers
  _Float16* xs = (_Float16*)smem;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int n_seg = (a.K + SEG - 1) / SEG;
  const int kpad = a.x_stride;
  for (int u = tid; u < MB * (kpad / 8); u += 1024) {
    const int m = u / (kpad / 8), k = 8 * (u - m * (kpad / 8));
    u4 v = u4{0, 0, 0, 0};
    if (k < a.K) v = *(const u4*)(a.X + (size_t)m * a.K + k);
    *(u4*)(xs + (size_t)m * kpad + k) = v;
  }
  __syncthreads();

  const int n_waves = gridDim.x * 16;
  const int first = __builtin_amdgcn_readfirstlane(blockIdx.x * 16 + wave);  // this wave's first row
  const int n_rows = first < a.N ? (a.N - first + n_waves - 1) / n_waves : 0;
  const int total = n_rows * n_seg;  // segments this wave reads, row after row
  if (total == 0) return;
  const _Float16* W = (const _Float16*)a.W;
  u4 ring[RS];
  int rq = 0;  // next segment to request (clamped to the last: requests past the end are ignored)
  auto request = [&](u4& slot) {
    const int c = min(rq, total - 1);
    const int ri = c / n_seg, seg = c - ri * n_seg;
    const int k = seg * SEG + 8 * lane;
    const bool ok = k < a.K;
    const u4* p = (const u4*)(W + (size_t)(first + ri * n_waves) * a.K + (ok ? k : 0));
    const u4 v = NT ? __builtin_nontemporal_load(p) : *p;
    const uint32_t keep = ok ? 0xFFFFFFFFu : 0u;  // lanes beyond K re-read the row's start and drop it
    slot = u4{v[0] & keep, v[1] & keep, v[2] & keep, v[3] & keep};
    rq++;
  };
#pragma unroll
  for (int q = 0; q < LR; q++) {
    request(ring[q]);
    __builtin_amdgcn_sched_barrier(0);
  }
  float acc[MB];
#pragma unroll
  for (int m = 0; m < MB; m++) acc[m] = 0.0f;
  int row = first, seg = 0;
  auto step = [&](u4& slot, u4& free_slot) {
    request(free_slot);
    __builtin_amdgcn_sched_barrier(0);
    const h8 w = __builtin_bit_cast(h8, slot);
    const _Float16* x = xs + seg * SEG + 8 * lane;
#pragma unroll
    for (int m = 0; m < MB; m++) {
      const h8 xv = *(const h8*)(x + (size_t)m * kpad);
#pragma unroll
      for (int q = 0; q < 4; q++) acc[m] = __builtin_amdgcn_fdot2(h2{w[2 * q], w[2 * q + 1]}, h2{xv[2 * q], xv[2 * q + 1]}, acc[m], false);
    }
    if (++seg == n_seg) {  // the row is complete: add its 64 lanes up and store
#pragma unroll
      for (int m = 0; m < MB; m++) {
        float v = acc[m];
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) v += __shfl_xor(v, d);
        if (lane == 0) a.Y[(size_t)m * a.N + row] = __builtin_bit_cast(uint16_t, (_Float16)v);
        acc[m] = 0.0f;
      }
      seg = 0;
      row += n_waves;
    }
  };
  int i = 0;
  for (; i + RS <= total; i += RS) {
#pragma unroll
    for (int q = 0; q < RS; q++) {
      step(ring[q], ring[(q + LR) % RS]);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int q = 0; q < RS - 1; q++)
    if (i + q < total) step(ring[q], ring[(q + LR) % RS]);
}

// Finish one strip with the complete tile of this workgroup's slice of K: times the scales, converted, stored; with
// K split over gk workgroups, through the workspace.
template <int MT>
__device__ __forceinline__ void finish_strip(const LinearArgs& a, int gk, int out_strip, f4 (&sum)[MT], const f4 sc, int lane) {
  if (a.gk > 1 && !exchange_tile<MT>(a, gk, out_strip, sum, lane)) return;
  store_tile_scaled<MT>(sum, sc, a, out_strip, lane);
}

// The Linear on packed weights.  A workgroup owns up to 16 neighbouring strips (spw of them,
// one resident round of workgroups; more strips than 16 x 256 just means more workgroups) and
// has S / spw wavefronts on each: a wavefront stays with its strip and takes every wps-th
// record of it, in step with all other wavefronts of the grid.  With the K-major packed layout
// the grid as a whole then reads one contiguous window of memory that moves through the
// matrix front to back (measured with bare read kernels under a realistic amount of per-record
// arithmetic: 10-20 % faster than strips that are read as separate streams).  A strip's
// partial tile stays in its wavefront's accumulator registers for the whole of K, also across
// the phases K is walked in when the activations M x K do not fit in LDS; at the end the wps
// tiles of a strip are added in wave order through LDS (deterministic, no atomics), scaled,
// converted and stored; a wavefront that is alone on its strip (wps = 1) finishes it straight
// from its accumulators.  Each wave keeps LR records in flight beside the one it is restoring
// (two with 16 wavefronts per workgroup, three with 8: the host decides which).
// QD (formats with side bits): the records are dealt to a strip's wavefronts in whole side groups,
// so that a group's side dword is loaded once per group and not once per record; used where the
// groups of a phase divide evenly enough among the wavefronts (the host decides).
// RAGGED: rows of X that are not 16-byte aligned (K % 8 != 0).  An instantiation of its own: with the choice made at
// run time the aligned launches of M = 16 and 32 took 5-10 % longer (4096 x 4096 FP4.25 at M = 32 13.4 -> 14.9 us).
template <int FMT, int MT, bool NT, bool GS, bool QD = false, int LR = 2, bool RAGGED = false>
__global__ void __launch_bounds__(1024) column_kernel(LinearArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int REC_K = Fmt<FMT>::REC_K, SG = Fmt<FMT>::SG, RS = LR + 1;
  // the side-group deal has a ring of four slots and two side registers: a request must stay within the group after
  // the one being multiplied
  static_assert(!QD || LR == 2 || (LR == 3 && SG == 4), "records ahead in the side-group deal");
  asm volatile("" ::"s"(a.W), "s"(a.scales), "s"(a.X), "s"(a.Y), "s"(a.M), "s"(a.N), "s"(a.K), "s"(a.n_rec), "s"(a.x_stride),
               "s"(a.x_region), "s"(a.x_shift), "s"(a.n_strips), "s"(a.spw), "s"(a.rc), "s"(a.gn), "s"(a.gk), "s"(a.wps));
  const int tid = threadIdx.x, lane = tid & 63, nthr = blockDim.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int S = nthr >> 6;
  // workgroup = (position g along N, slice gk of K); without a split the grid is all along N
  const int G = a.gn;
  const int gk = a.gk > 1 ? (int)(blockIdx.x / (unsigned)G) : 0;
  const int g = (int)blockIdx.x - gk * G;
  const int s_first = g * a.spw;                      // this workgroup's strips: s_first .. s_first + ns - 1
  const int ns = min(a.spw, a.n_strips - s_first);    // >= 1
  const int wps = a.wps;                              // wavefronts per strip
  const int wj = (int)((unsigned)wave / (unsigned)wps), wk = wave - wj * wps;  // this wave: strip wj of the workgroup, lane wk of its K deal
  const bool has_strip = wj < ns && wk < a.wpa;
  const int strip = s_first + (wj < ns ? wj : 0);
  // records [rec_lo, rec_hi) of every strip are this workgroup's slice of K
  const int rec_lo = a.gk > 1 ? (int)((unsigned)(gk * a.n_rec) / (unsigned)a.gk) : 0;
  const int rec_hi = a.gk > 1 ? (int)((unsigned)((gk + 1) * a.n_rec) / (unsigned)a.gk) : a.n_rec;
  const int RC = a.rc;  // records per strip in one phase of K
  const int mc = min(a.M, 16);  // activation rows of an MFMA tile that exist
  _Float16* xs = (_Float16*)smem;
  f4* parts = (f4*)(smem + (size_t)a.x_region * 2);  // [spw][wps][MT][4 K-quarters][mc]
  const int m_lo = lane & 15, kq = lane >> 4;
  const int lane_off = (REC_K / 4) * kq;
  // lanes whose activation row does not exist read row 0: they only feed output columns never stored
  const _Float16* x0 = xs + (m_lo < a.M ? m_lo : 0) * a.x_stride + lane_off;
  const _Float16* x1 = xs + (m_lo + 16 < a.M ? m_lo + 16 : 0) * a.x_stride + lane_off;
  const int part_f4 = MT * 4 * mc;  // f4 per parked tile

  const int total_units = a.M << a.x_shift;
  const int units_per_pass = nthr * XUnit<FMT>::XU;
  const bool wave_has_x = (!RAGGED || a.K >= 8) && wave * 64 < total_units;  // wave-uniform
  const int chunk_k = RC * REC_K;
  // Scales of the strip this wave finishes (wave w finishes strip w of the workgroup): requested first, kept as raw
  // bits until the epilogue.  (With one scale per run of input channels, GS, the scales travel with the records.)
  ScaleBits scale0_bits = {{0x3C00, 0x3C00, 0x3C00, 0x3C00}};
  if constexpr (!GS) scale0_bits = load_scale_bits<FMT>(a, min(s_first + min(wave, ns - 1), a.n_strips - 1), lane);
  __builtin_amdgcn_sched_barrier(0);

  f4 acc[MT];
#pragma unroll
  for (int i = 0; i < MT; i++) acc[i] = f4{0, 0, 0, 0};

  // K is walked in phases of RC records per strip (one phase when all activations fit in LDS).
  for (int rec_base = rec_lo; rec_base < rec_hi; rec_base += RC) {
    const int n_rec = min(RC, rec_hi - rec_base);                                    // records per strip in this phase
    const int cnt = (has_strip && wk < n_rec) ? (n_rec - wk + wps - 1) / wps : 0;  // records of this wave
    if (rec_base > rec_lo) __syncthreads();  // everyone is done with the previous phase's activations
    const int k0 = rec_base * REC_K;

    // Activations: units beyond the first pass (large M) and unaligned rows are staged by loops
    // that run to completion; the first pass is only requested here and stored behind the
    // head of the weight stream, so both are in flight together.
    XRegs<FMT> xr;
    if (!RAGGED || a.K >= 8) {
      for (int u0 = units_per_pass; u0 < total_units; u0 += nthr * XUnit<FMT>::XB) {
        XRegs<FMT, XUnit<FMT>::XB> xb;
        x_load<RAGGED>(xb, a, k0, chunk_k, u0, tid, nthr);
        x_store<RAGGED>(xb, xs, a, k0, chunk_k, u0, tid, nthr);
      }
      if (wave_has_x) x_load<RAGGED>(xr, a, k0, chunk_k, 0, tid, nthr);
    } else {
      stage_x_short<FMT>(xs, a, k0, chunk_k, tid, nthr);
    }
    __builtin_amdgcn_sched_barrier(0);

    if constexpr (QD) {
      // Side groups dealt whole: the wave's records are its groups wk, wk + wpa, ... of the phase, member by
      // member.  Two groups per unrolled round, so that the ring slot of a record (its number mod 4), the side
      // register of its group (the group's number mod 2) and its place in the side dword are all fixed in the
      // code.  LR = 2 records ahead as above; a group's side dword is requested with its first record.
      constexpr int UN = 2 * SG;
      const int n_grp = (n_rec + SG - 1) / SG;  // the phase starts on a group boundary; a last group may run into the padding records
      const int wpa = a.wpa;
      const int cnt_g = (has_strip && wk < n_grp) ? (n_grp - wk + wpa - 1) / wpa : 0;
      const int total_e = cnt_g * SG, e_last = max(total_e - 1, 0);
      const int g_first = cnt_g > 0 ? wk : 0;
      LaneRec<FMT> ring[4];
      uint32_t side[2] = {0, 0};
      // e-th record of this wave (clamped to its last): group g_first + (e / SG) * wpa, member e % SG
      auto request = [&](int e, LaneRec<FMT>& slot, uint32_t& side_reg, bool with_side) {
        e = min(e, e_last);
        const int grp = rec_base / SG + g_first + (e / SG) * wpa;
        const uint8_t* unit = a.W + ((size_t)grp * a.n_strips + strip) * Fmt<FMT>::UNIT;
        load_lane_rec<FMT, NT, false>(slot, unit + (e % SG) * Fmt<FMT>::CB, nullptr, lane);
        if (with_side) {
          const uint32_t* sp = (const uint32_t*)(unit + SG * Fmt<FMT>::CB) + lane;
          side_reg = NT ? __builtin_nontemporal_load(sp) : *sp;
        }
      };
#pragma unroll
      for (int q = 0; q < LR; q++) {
        request(q, ring[q], side[(q / SG) & 1], q % SG == 0);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (wave_has_x) x_store<RAGGED>(xr, xs, a, k0, chunk_k, 0, tid, nthr);
      __syncthreads();

      int rel = g_first * SG;  // first record of the group being multiplied, relative to the phase
      auto round_of = [&](int b, auto n_steps) {
#pragma unroll
        for (int u = 0; u < decltype(n_steps)::value; u++) {
          request(b + u + LR, ring[(u + LR) & 3], side[((u + LR) / SG) & 1], (u + LR) % SG == 0);
          __builtin_amdgcn_sched_barrier(0);
          LaneRec<FMT> cur = ring[u & 3];
          cur.t = side[(u / SG) & 1];
          const int kk = (rel + u % SG) * REC_K;
          mac_rec<FMT, MT>(cur, x0 + kk, x1 + kk, acc, 8 * Fmt<FMT>::SIDE * (u % SG));
          if (u % SG == SG - 1) rel += wpa * SG;
          __builtin_amdgcn_sched_barrier(0);
        }
      };
      int b = 0;
      for (; b + UN <= total_e; b += UN) round_of(b, std::integral_constant<int, UN>{});
      if (b < total_e) round_of(b, std::integral_constant<int, SG>{});  // an odd last group
    } else {
      // LR records are in flight while a record is being restored: the ring has one slot more,
      // and a step first requests the record LR places ahead into the slot freed by the step
      // before, then works on its own.  The request cursor stops at the wave's last record (a
      // wave without records requests, and ignores, the phase's first record of its strip).
      struct Slot {
        LaneRec<FMT> r;
        us4 gs;  // GS: the scales of this lane's four output channels for the record's run
      };
      Slot ring[RS];
      int pr = rec_base + (cnt > 0 ? wk : 0);                       // record the next request fetches
      const int pr_last = rec_base + (cnt > 0 ? wk + (cnt - 1) * wps : 0);
      auto request = [&](Slot& slot) {
        load_rec<FMT, NT>(slot.r, a, strip, pr, lane);
        if constexpr (GS)  // 8 bytes, the same for the 16 lanes of a K-quarter; cached: a run spans many records
          slot.gs = *(const us4*)(a.scales + ((size_t)strip * a.n_sg + (pr >> a.sg_shift)) * 16 + 4 * kq);
        pr = min(pr + wps, pr_last);
      };
  #pragma unroll
      for (int q = 0; q < LR; q++) {
        request(ring[q]);
        __builtin_amdgcn_sched_barrier(0);  // issue in ring order: the oldest load is the first one needed
      }
      if (wave_has_x) x_store<RAGGED>(xr, xs, a, k0, chunk_k, 0, tid, nthr);
      __syncthreads();

      // One record: request the one LR ahead, restore, multiply, move on by wps records.
      int cr = wk;  // record being multiplied, relative to the phase
      auto step = [&](Slot& slot, Slot& free_slot) {
        request(free_slot);
        __builtin_amdgcn_sched_barrier(0);
        const int side_shift = 8 * Fmt<FMT>::SIDE * ((rec_base + cr) & (SG - 1));
        if constexpr (GS) {  // the record's own tile, times its run's scales (Eq. 2), then into the sum
          f4 t[MT];
  #pragma unroll
          for (int i = 0; i < MT; i++) t[i] = f4{0, 0, 0, 0};
          mac_rec<FMT, MT>(slot.r, x0 + cr * REC_K, x1 + cr * REC_K, t, side_shift);
          f4 sc;
  #pragma unroll
          for (int r = 0; r < 4; r++) sc[r] = (float)__builtin_bit_cast(_Float16, (uint16_t)slot.gs[r]);
  #pragma unroll
          for (int i = 0; i < MT; i++) acc[i] += t[i] * sc;
        } else {
          mac_rec<FMT, MT>(slot.r, x0 + cr * REC_K, x1 + cr * REC_K, acc, side_shift);
        }
        cr += wps;
      };
      int i = 0;
      for (; i + RS <= cnt; i += RS) {
  #pragma unroll
        for (int q = 0; q < RS; q++) {
          step(ring[q], ring[(q + LR) % RS]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
  #pragma unroll
      for (int q = 0; q < RS - 1; q++)
        if (i + q < cnt) step(ring[q], ring[(q + LR) % RS]);
    }
  }

  // Finish strip j of the workgroup with its complete tile of this workgroup's slice of K.
  auto finish = [&](int j, f4 (&sum)[MT]) {
    const int out_strip = s_first + j;
    f4 sc;
    if constexpr (GS)
      sc = f4{kTwo14, kTwo14, kTwo14, kTwo14};
    else
      sc = j == wave ? scales_from_bits(scale0_bits, kTwo14) : load_scales<FMT>(a, out_strip, lane);
    finish_strip<MT>(a, gk, out_strip, sum, sc, lane);
  };
  // A wavefront that is alone on its strip finishes it straight from its accumulators.
  if (wps == 1) {
    if (wj < ns) finish(wj, acc);
    return;
  }
  // Otherwise one wave per strip adds the wps tiles of the strip in wave order, through LDS.
  if (wj < ns && m_lo < mc) {  // idle wavefronts of a strip leave a tile of zeros
    f4* t = parts + (size_t)(wj * wps + wk) * part_f4 + kq * mc + m_lo;
#pragma unroll
    for (int i = 0; i < MT; i++) t[i * 4 * mc] = acc[i];
  }
  __syncthreads();
  for (int j = wave; j < ns; j += S) {
    f4 sum[MT];
#pragma unroll
    for (int t = 0; t < MT; t++) sum[t] = f4{0, 0, 0, 0};
    if (m_lo < mc) {
      const f4* t0 = parts + (size_t)j * wps * part_f4 + kq * mc + m_lo;
      for (int w = 0; w < wps; w++) {
#pragma unroll
        for (int t = 0; t < MT; t++) sum[t] += t0[(size_t)w * part_f4 + t * 4 * mc];
      }
    }
    finish(j, sum);
  }
}

// The Linear on packed weights where a workgroup owns more strips than it has wavefronts: eight wavefronts, each
// alone on NS strips of the workgroup (wave w on strips w, w + wn, ...; wn = a.wpa wavefronts own strips), which it
// walks record by record side by side (record r of its first strip, record r of its second, record r + 1 ...), one
// accumulator tile per strip, three records ahead in a ring of four.  All strips of the workgroup are still read
// at the same record index at the same time (the contiguous window of the column kernel), the activations are
// staged as there, and every strip is finished straight from its wavefront's accumulators: no tiles in LDS, no
// barrier after the last record.  For the formats whose records carry no side groups (with the side groups of two
// strips dealt in turn FP4.25 was 1-3 % slower than with sixteen wavefronts on one strip each: measured, not kept).
template <int FMT, int MT, bool NT, int NS, bool RAGGED = false>
__global__ void __launch_bounds__(512) multi_kernel(LinearArgs a) {
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int REC_K = Fmt<FMT>::REC_K, SG = Fmt<FMT>::SG, LR = 3;
  static_assert(NS == 2 || NS == 4, "strips per wavefront: the ring of four must hold whole rounds of them");
  asm volatile("" ::"s"(a.W), "s"(a.scales), "s"(a.X), "s"(a.Y), "s"(a.M), "s"(a.N), "s"(a.K), "s"(a.n_rec), "s"(a.x_stride),
               "s"(a.x_region), "s"(a.x_shift), "s"(a.n_strips), "s"(a.spw), "s"(a.rc), "s"(a.gn), "s"(a.gk), "s"(a.wpa));
  const int tid = threadIdx.x, lane = tid & 63, nthr = blockDim.x;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = a.gn;
  const int gk = a.gk > 1 ? (int)(blockIdx.x / (unsigned)G) : 0;
  const int g = (int)blockIdx.x - gk * G;
  const int s_first = g * a.spw;
  const int ns = min(a.spw, a.n_strips - s_first);  // >= 1
  const int wn = a.wpa;                             // wavefronts that own strips
  const bool has_strip = wave < wn && wave < ns;
  int sidx[NS];    // this wave's strips (those that do not exist stand for the workgroup's last: read, never finished)
  bool valid[NS];
#pragma unroll
  for (int i = 0; i < NS; i++) {
    valid[i] = wave < wn && wave + i * wn < ns;
    sidx[i] = s_first + min(wave + i * wn, ns - 1);
  }
  const int rec_lo = a.gk > 1 ? (int)((unsigned)(gk * a.n_rec) / (unsigned)a.gk) : 0;
  const int rec_hi = a.gk > 1 ? (int)((unsigned)((gk + 1) * a.n_rec) / (unsigned)a.gk) : a.n_rec;
  const int RC = a.rc;
  _Float16* xs = (_Float16*)smem;
  const int m_lo = lane & 15, kq = lane >> 4;
  const int lane_off = (REC_K / 4) * kq;
  const _Float16* x0 = xs + (m_lo < a.M ? m_lo : 0) * a.x_stride + lane_off;
  const _Float16* x1 = xs + (m_lo + 16 < a.M ? m_lo + 16 : 0) * a.x_stride + lane_off;
  const int total_units = a.M << a.x_shift;
  const int units_per_pass = nthr * XUnit<FMT>::XU;
  const bool wave_has_x = (!RAGGED || a.K >= 8) && wave * 64 < total_units;  // wave-uniform
  const int chunk_k = RC * REC_K;
  ScaleBits sb[NS];
#pragma unroll
  for (int i = 0; i < NS; i++) sb[i] = load_scale_bits<FMT>(a, sidx[i], lane);
  __builtin_amdgcn_sched_barrier(0);

  f4 acc[NS][MT];
#pragma unroll
  for (int i = 0; i < NS; i++)
#pragma unroll
    for (int t = 0; t < MT; t++) acc[i][t] = f4{0, 0, 0, 0};

  for (int rec_base = rec_lo; rec_base < rec_hi; rec_base += RC) {
    const int n_rec = min(RC, rec_hi - rec_base);
    if (rec_base > rec_lo) __syncthreads();  // everyone is done with the previous phase's activations
    const int k0 = rec_base * REC_K;
    XRegs<FMT> xr;
    if (!RAGGED || a.K >= 8) {
      for (int u0 = units_per_pass; u0 < total_units; u0 += nthr * XUnit<FMT>::XB) {
        XRegs<FMT, XUnit<FMT>::XB> xb;
        x_load<RAGGED>(xb, a, k0, chunk_k, u0, tid, nthr);
        x_store<RAGGED>(xb, xs, a, k0, chunk_k, u0, tid, nthr);
      }
      if (wave_has_x) x_load<RAGGED>(xr, a, k0, chunk_k, 0, tid, nthr);
    } else {
      stage_x_short<FMT>(xs, a, k0, chunk_k, tid, nthr);
    }
    __builtin_amdgcn_sched_barrier(0);

    LaneRec<FMT> ring[4];
    {
      // records e = 0 .. NS * n_rec - 1 of the phase: strip e % NS, record e / NS
      const int total_e = has_strip ? NS * n_rec : 0;
      int qr = 0;  // record of the next request, relative to the phase (stops at the last)
      auto request = [&](LaneRec<FMT>& slot, int i) {
        load_rec<FMT, NT>(slot, a, sidx[i], rec_base + min(qr, n_rec - 1), lane);
        if (i == NS - 1) qr++;
      };
#pragma unroll
      for (int q = 0; q < LR; q++) {
        request(ring[q], q % NS);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (wave_has_x) x_store<RAGGED>(xr, xs, a, k0, chunk_k, 0, tid, nthr);
      __syncthreads();
      int cr = 0;  // record being multiplied, relative to the phase
      auto step = [&](auto uc) {
        constexpr int u = decltype(uc)::value;
        request(ring[(u + LR) & 3], (u + LR) % NS);
        __builtin_amdgcn_sched_barrier(0);
        const int side_shift = 8 * Fmt<FMT>::SIDE * ((rec_base + cr) & (SG - 1));
        mac_rec<FMT, MT>(ring[u & 3], x0 + cr * REC_K, x1 + cr * REC_K, acc[u % NS], side_shift);
        if (u % NS == NS - 1) cr++;
        __builtin_amdgcn_sched_barrier(0);
      };
      int e = 0;
      for (; e + 4 <= total_e; e += 4) {
        step(std::integral_constant<int, 0>{});
        step(std::integral_constant<int, 1>{});
        step(std::integral_constant<int, 2>{});
        step(std::integral_constant<int, 3>{});
      }
      if (e < total_e) {  // NS = 2 and an odd number of records: one more of each strip
        step(std::integral_constant<int, 0>{});
        step(std::integral_constant<int, 1>{});
      }
    }
  }

#pragma unroll
  for (int i = 0; i < NS; i++)
    if (valid[i]) finish_strip<MT>(a, gk, sidx[i], acc[i], scales_from_bits(sb[i], kTwo14), lane);
}

// Restore a whole packed matrix to row-major fp16: one wavefront per record, the records of a strip on neighbouring
// wavefronts.  Bound by the stores (2 bytes out per 0.5-0.75 in).  A lane owns a K-quarter of a row, 48 or 64 bytes of
// the result, so the record goes through the wavefront's own LDS tile and leaves it row by row in 16-byte stores, each
// row of the record one contiguous 192- or 256-byte run.  28672 x 4096 FP4.25: 55 us, 5.4 TB/s, what a copy of 1 GiB reaches (element by element,
// two bytes at a stride of a K-quarter per lane: 551 us).
constexpr int kDequantWaves = 4;  // of a workgroup
template <int FMT>
__global__ void __launch_bounds__(64 * kDequantWaves) dequant_kernel(const uint8_t* W, const uint16_t* scales, uint16_t* out, int N, int K,
                                                                     int n_rec, int64_t total_recs, int scaled, int n_sg, int sg_shift) {
  typedef _Float16 h2 __attribute__((ext_vector_type(2)));
  constexpr int SG = Fmt<FMT>::SG, REC_K = Fmt<FMT>::REC_K, PB = Fmt<FMT>::PB, LANE_K = REC_K / 4, PIECES = REC_K / 8;
  constexpr int TILE = REC_K + 8;  // halfs between the rows of a tile: neighbouring rows start 16 bytes apart in the banks
  __shared__ __attribute__((aligned(16))) uint16_t tiles[kDequantWaves][16 * TILE];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t rec_id = (int64_t)blockIdx.x * kDequantWaves + wave;
  if (rec_id >= total_recs) return;
  const int strip = (int)(rec_id / n_rec), rec = (int)(rec_id - (int64_t)strip * n_rec);
  const int64_t n_strips = (N + 15) / 16;
  const uint8_t* unit = W + ((size_t)(rec / SG) * n_strips + strip) * Fmt<FMT>::UNIT;
  LaneRec<FMT> r;
  load_lane_rec<FMT, true>(r, unit + (rec % SG) * Fmt<FMT>::CB, unit + SG * Fmt<FMT>::CB, lane);
  // one scale per row (sg_shift < 0) or per run of 2^sg_shift records: [strip][run][row in strip]
  _Float16 s = 1;
  if (scaled) {
    const int n = min(strip * 16 + (lane & 15), N - 1);  // rows beyond N are never stored
    s = __builtin_bit_cast(_Float16, sg_shift < 0 ? scales[n] : scales[((size_t)strip * n_sg + (rec >> sg_shift)) * 16 + (lane & 15)]);
  }
  uint32_t o[4 * Fmt<FMT>::N_MFMA];
  restore_rec<FMT>(r, 8 * Fmt<FMT>::SIDE * (rec % SG), o);
  // Magnitudes times 2^14 (exact) times the scale (the exact product, rounded once); the sign bit apart, so that a
  // negative zero code keeps it.
#pragma unroll
  for (int m = 0; m < 4 * Fmt<FMT>::N_MFMA; m++) {
    const h2 v = __builtin_bit_cast(h2, o[m] & 0x7FFF7FFFu) * h2{(_Float16)kTwo14, (_Float16)kTwo14} * h2{s, s};
    o[m] = __builtin_bit_cast(uint32_t, v) | (o[m] & 0x80008000u);
  }
  // from operand order into input-channel order, into the tile
  uint16_t* tile = tiles[wave];
  u4* mine = (u4*)(tile + (lane & 15) * TILE + (lane >> 4) * LANE_K);
#pragma unroll
  for (int d = 0; d < LANE_K / 8; d++) {
    u4 v;
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const int j = 8 * d + 2 * e, blk = j / PB * PB;  // input channels j, j + 1 of the lane's K-quarter
      v[e] = pick2(o + blk / 2, channel_slot<FMT>(j - blk), channel_slot<FMT>(j + 1 - blk));
    }
    mine[d] = v;
  }
  __builtin_amdgcn_wave_barrier();  // the tile is this wavefront's own, LDS serves it in order
  const int k0 = rec * REC_K;
#pragma unroll
  for (int i = 0; i < PIECES / 4; i++) {
    const int q = i * 64 + lane, row = q / PIECES, p = q - row * PIECES;  // 8 channels of one row
    const u4 v = *(const u4*)(tile + row * TILE + 8 * p);
    const int n = strip * 16 + row, k = k0 + 8 * p;
    if (n < N && k < K) {
      uint16_t* dst = out + (size_t)n * K + k;
      if (k + 8 <= K) {
        __builtin_memcpy(dst, &v, 16);  // rows start anywhere where K is no multiple of 8: one unaligned store
      } else {
#pragma unroll
        for (int e = 0; e < 7; e++)
          if (e < K - k) dst[e] = (uint16_t)(v[e >> 1] >> (16 * (e & 1)));
      }
    }
  }
}

// Measurement aid: reads n_rec records of 1 KiB and discards them.  Record r goes to
// wavefront r mod (all wavefronts of the grid), two records in flight per wave: the
// fastest read order found on this GPU, the ceiling the Linear kernels are compared with.
__global__ void __launch_bounds__(1024) read_probe_kernel(const u4* __restrict__ p, int64_t n_rec, uint32_t* sink) {
  const int lane = threadIdx.x & 63;
  const int S = blockDim.x >> 6;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t first = (int64_t)blockIdx.x * S + wave, step = (int64_t)gridDim.x * S;
  // nothing to read (the launch-floor mode) or no record for this wave: no load at all
  if (first >= n_rec) return;
  const int64_t last = n_rec - 1;  // >= 0 here; every index below is clamped into [0, last]
  u4 ring[2];
  uint32_t acc = 0;
#pragma unroll
  for (int i = 0; i < 2; i++) ring[i] = __builtin_nontemporal_load(p + min(first + i * step, last) * 64 + lane);
  for (int64_t r = first; r < n_rec; r += 2 * step) {
#pragma unroll
    for (int i = 0; i < 2; i++) {
      const u4 v = ring[i];
      ring[i] = __builtin_nontemporal_load(p + min(r + (i + 2) * step, last) * 64 + lane);
      if (r + i * step < n_rec) acc ^= v[0] ^ v[1] ^ v[2] ^ v[3];
    }
  }
  if (acc == 0x9E3779B9u && sink) sink[0] = acc;  // keeps the loads alive; practically never true
}

// ---- host-side launch logic -------------------------------------------------
// activations are staged in units of one permutation block
int x_unit(int fmt) { return fmt == FMT_FP16 ? 8 : ams::kFormats[fmt].perm_block; }

bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

constexpr int kNumCU = 256;             // MI355X compute units
constexpr int kStreamLdsMax = kLdsMaxBytes;  // one workgroup per compute unit: all of it (measured: the phases of K this saves pay)

struct StreamPlan {
  bool ok;
  int S, lr, spw, grid, rc, x_shift, x_stride, x_region, red_slots;
  size_t lds;
};

// Launch shape of the streaming kernel: one workgroup of 16 wavefronts per CU, each
// owning an equal run of whole strips; K is walked in as few phases as the LDS allows
// (activations of a phase: M x rc records; plus the waves' tile slots).
StreamPlan make_stream_plan(int fmt, int M, int64_t n_strips, int n_rec, int rec_k) {
  StreamPlan p;
  const int mt = M > 16 ? 2 : 1;
  // strips per workgroup: one resident round, but at most 32 (a wave parks one tile per strip it touches)
  p.spw = (int)std::min<int64_t>(32, (n_strips + kNumCU - 1) / kNumCU);
  p.grid = (int)((n_strips + p.spw - 1) / p.spw);
  p.ok = false;
  for (int n_phase = 1; n_phase <= n_rec; n_phase++) {
    const int rc = (n_rec + n_phase - 1) / n_phase;
    if (n_phase > 1 && rc == (n_rec + n_phase - 2) / (n_phase - 1)) continue;  // same rc as before
    const int64_t P = (int64_t)p.spw * rc;
    const int S = (int)std::min<int64_t>(16, std::max<int64_t>(1, P));
    const int per_wave_max = (int)((P + S - 1) / S);
    const int slots = (per_wave_max - 1) / rc + 2;
    const int x_stride = rc * rec_k + 8;  // +8 halfs: consecutive rows start 16 bytes apart in the banks
    const size_t lds = (size_t)M * x_stride * 2 + (size_t)S * slots * mt * 64 * 16;
    if (lds > (size_t)kStreamLdsMax) continue;
    p.ok = true;
    p.rc = rc;
    p.S = S;
    p.red_slots = slots;
    p.x_stride = x_stride;
    p.x_region = M * x_stride;
    p.lds = lds;
    // measured on the Llama-8B/70B shapes: deeper rings only lengthen the drain at the end of the stream
    p.lr = fmt == FMT_FP16 ? 2 : 4;  // the baseline's records are four times larger
    while (p.lr > 2 && p.lr > per_wave_max) p.lr /= 2;
    const int units = rc * rec_k / x_unit(fmt);
    p.x_shift = 0;
    while ((1 << p.x_shift) < units) p.x_shift++;
    break;
  }
  return p;
}

struct SweepPlan {
  bool ok;
  int S, lr, spw, grid, gn, gk, wps, rc, x_shift, x_stride, x_region;
  size_t lds;
};

// Launch shape of the sweeping kernel: one resident round of workgroups of up to 16
// wavefronts; LDS holds one parked tile per (strip, wave) and the activations of one
// phase of K, in as few phases as fit.
// any_shape: this kernel must take the shape (no other kernel can): strips per workgroup
// are capped so that the parked tiles fit, whatever number of rounds and phases that takes.
// gk > 1: K is cut in gk slices, each with its own kNumCU / gk workgroups along N.
SweepPlan make_sweep_plan(int fmt, int M, int64_t n_strips, int n_rec_all, int rec_k, bool any_shape = false, int gk = 1) {
  SweepPlan p;
  const int mt = M > 16 ? 2 : 1;
  const int mc = std::min(M, 16);
  p.ok = false;
  p.gk = gk;
  if (!any_shape && n_strips > (int64_t)kNumCU * 64) return p;
  const int n_rec = (n_rec_all + gk - 1) / gk;  // records of the longest slice
  const int wg_along_n = kNumCU / gk;
  p.spw = (int)((n_strips + wg_along_n - 1) / wg_along_n);
  const size_t tile_bytes = (size_t)mt * 4 * mc * 16;  // one parked tile
  if (any_shape) p.spw = (int)std::max<int64_t>(1, std::min<int64_t>(p.spw, (48 * 1024) / tile_bytes));
  p.gn = (int)((n_strips + p.spw - 1) / p.spw);
  p.grid = p.gn * gk;
  // The baseline's records are four times larger (one in flight per wave).  Measured: at M <= 4 with every
  // compute unit busy it reads 8-14 % faster from 8 wavefronts with two records in flight each (the packed
  // formats do not: equal at M = 1, slower from M = 8).
  const bool few_waves = fmt == FMT_FP16 && M <= 4 && gk == 1 && !any_shape && n_strips >= kNumCU && p.spw <= 16;
  p.S = (int)std::min<int64_t>(few_waves ? 8 : 16, (int64_t)p.spw * (n_rec_all / gk));  // n_rec_all / gk: the shortest slice
  if (p.S < 1) return p;
  p.lr = fmt == FMT_FP16 ? (few_waves ? 2 : 1) : 2;
  // waves per strip: all of them unless the parked tiles (one per strip and wave of its group)
  // would take more than 48 KB; never fewer than leaves every group of waves a strip
  p.wps = p.S;
  if (p.S == 16)
    while (p.wps > 1 && (size_t)p.spw * p.wps * tile_bytes > 48 * 1024 && 16 / (p.wps / 2) <= p.spw) p.wps /= 2;
  const size_t parts = (size_t)p.spw * p.wps * tile_bytes;
  for (int n_phase = 1; n_phase <= (any_shape ? n_rec : 8) && n_phase <= n_rec; n_phase++) {
    const int rc = (n_rec + n_phase - 1) / n_phase;
    const int x_stride = rc * rec_k + 8;  // +8 halfs: consecutive rows start 16 bytes apart in the banks
    const size_t lds = (size_t)M * x_stride * 2 + parts;
    if (lds > (size_t)kStreamLdsMax) continue;
    // measured: with many parked tiles and more than four phases (two for the baseline's larger records) the
    // contiguous-piece kernel is faster
    if (!any_shape && n_phase > (fmt == FMT_FP16 ? 2 : 4) && parts > 32 * 1024) break;
    p.ok = true;
    p.rc = rc;
    p.x_stride = x_stride;
    p.x_region = M * x_stride;
    p.lds = lds;
    const int units = rc * rec_k / x_unit(fmt);
    p.x_shift = 0;
    while ((1 << p.x_shift) < units) p.x_shift++;
    break;
  }
  return p;
}

struct ColumnPlan {
  int S, spw, grid, gn, gk, wps, rc, n_phase, x_shift, x_stride, x_region;
  bool qd;  // records dealt in whole side groups
  int wpa;  // wavefronts of a strip that take records (= wps unless fewer divide the side groups evenly)
  int lr;   // records a wavefront keeps in flight beside the one it restores
  int ns;   // strips a wavefront owns alone (multi_kernel; 1: column_kernel); then wpa = wavefronts that own strips
  bool slice;  // slice_kernel: the wavefronts share K and take every record of all spw strips; S, spw, grid, gn, gk, lr and lds hold
  int variant;  // slice_kernel's
  int rows, row_tiles;  // slice_kernel: staged rows of X per workgroup, workgroups that share the rows
  size_t lds;
};

// Launch shape of the packed formats' kernel for S wavefronts per workgroup that keep lr records in flight each: up
// to 16 neighbouring strips per workgroup (one resident round of workgroups where the matrix allows it), S / strips
// wavefronts on each strip; LDS holds the activations of one phase of K, in as few phases as fit,
// and one tile per wavefront for the final sum.  Every shape the entry points accept gets a plan.
// gk > 1: K is cut in gk slices, each with its own kNumCU / gk workgroups along N.
// allow_qd: the caller's variant can deal whole side groups (not with one scale per run of input channels).
ColumnPlan column_plan_for(int S, int lr, int fmt, int M, int64_t n_strips, int n_rec_all, int rec_k, int gk, bool allow_qd,
                           int ns = 1) {
  ColumnPlan p;
  p.ns = ns;
  p.slice = false;
  p.variant = kSlicePlain;
  p.rows = M;
  p.row_tiles = 1;
  const int sg = ams::side_group(ams::kFormats[fmt]);
  const int mt = M > 16 ? 2 : 1;
  const int mc = std::min(M, 16);
  p.gk = gk;
  p.S = S;
  p.lr = lr;
  const int n_rec = (n_rec_all + gk - 1) / gk;  // records of the longest slice
  const int wg_along_n = kNumCU / gk;
  p.spw = (int)std::min<int64_t>(16, (n_strips + wg_along_n - 1) / wg_along_n);
  p.gn = (int)((n_strips + p.spw - 1) / p.spw);
  p.grid = p.gn * gk;
  p.wps = ns > 1 ? 1 : p.S / p.spw;
  const size_t parts = ns > 1 ? 0 : (size_t)p.spw * p.wps * mt * 4 * mc * 16;  // at most 32 KiB
  // Whole side groups per wavefront where that divides the work evenly enough: the phases then start on group
  // boundaries, and every wavefront of a strip must get (nearly) the same number of groups.
  p.qd = false;
  for (int n_phase = 1;; n_phase++) {
    int rc = (n_rec + n_phase - 1) / n_phase;
    bool qd = allow_qd && sg > 1 && gk == 1;
    int wpa = p.wps;
    if (qd) {
      // the most wavefronts per strip, at least 7 of 8 of them, among which the groups divide within 20 %.  Measured
      // on eleven shapes and four formats: a wavefront with a fifth more records than the average costs less than
      // a side dword loaded with every record (each of a group's records is then read by another wavefront, and
      // each loads the group's 256 bytes of side bits again: 2-14 % slower), while leaving more than an eighth of
      // the wavefronts without records to make the groups divide costs more than it gains (up to 9 % slower)
      const int rcq = (rc + sg - 1) / sg * sg;
      const int groups = rcq / sg;
      qd = false;
      if ((size_t)M * (rcq * rec_k + 8) * 2 + parts <= (size_t)kLdsMaxBytes)
        for (int w = p.wps; w * 8 >= p.wps * 7 && w >= 1 && !qd; w--)
          if (groups >= w && (groups + w - 1) / w * w * 100 <= groups * 120) qd = true, wpa = w;
      if (qd) rc = rcq;
    }
    const int x_stride = rc * rec_k + 8;  // +8 halfs: consecutive rows start 16 bytes apart in the banks
    const size_t lds = (size_t)M * x_stride * 2 + parts;
    if (lds > (size_t)kLdsMaxBytes && rc > 1) continue;  // one record per phase always fits (32 rows x 136 halfs)
    p.qd = qd;
    p.wpa = ns > 1 ? (p.spw + ns - 1) / ns : wpa;
    p.rc = rc;
    p.n_phase = (n_rec + rc - 1) / rc;
    p.x_stride = x_stride;
    p.x_region = M * x_stride;
    p.lds = lds;
    const int units = rc * rec_k / x_unit(fmt);
    p.x_shift = 0;
    while ((1 << p.x_shift) < units) p.x_shift++;
    break;
  }
  return p;
}

// allow_qd: the caller's variant can deal whole side groups (not with one scale per run of input channels).
// allow_deep: the caller has the kernel with three records ahead (non-temporal loads, one scale per row).
ColumnPlan make_column_plan(int fmt, int M, int64_t n_strips, int n_rec_all, int rec_k, int gk = 1, bool allow_qd = true,
                            bool allow_deep = true) {
  const ColumnPlan p = column_plan_for(16, 2, fmt, M, n_strips, n_rec_all, rec_k, gk, allow_qd);
  // Eight wavefronts with three records ahead instead of sixteen with two: fewer wavefronts contend for the VALU
  // and nearly the same bytes are in flight.  Measured on fourteen shapes: formats whose records carry no side
  // groups are 1-7 % faster where the workgroups fill the chip, at least seven of the eight wavefronts get a strip
  // or an equal share of one, and a wavefront's stream is long enough to amortise the deeper ring's start; slower
  // elsewhere, and slower at larger batches (half the threads stage the activations) except where a wavefront is
  // alone on its strip and needs no sum through LDS at the end (up to a batch of 8).  With the side groups dealt
  // whole only that last case gains: FP4.25 0-8 % (kept), FP4.33 -4 % at K = 4096 and +3 % at K = 8192 (not kept).
  const int sg = ams::side_group(ams::kFormats[fmt]);
  const int n_rec = (n_rec_all + gk - 1) / gk;
  // More strips than eight wavefronts: two strips per wavefront, side by side (70B gate/up 50.8 -> 48.5 us, the
  // 128256 x 4096 vocabulary projection 55.1 -> 54.5, the same at K = 8192 +- 0; batches up to 8 measured).
  if (allow_deep && sg == 1 && gk == 1 && p.spw >= 9 && p.grid >= kNumCU * 7 / 8 && n_rec >= 8 && M <= 8)
    return column_plan_for(8, 3, fmt, M, n_strips, n_rec_all, rec_k, gk, allow_qd, 2);
  const int active = p.spw <= 8 ? (8 / p.spw) * p.spw : 0;  // of eight wavefronts, those that get records
  if (!allow_deep || gk != 1 || active < 7 || p.grid < kNumCU * 7 / 8 || (int64_t)n_rec * p.spw < 16 * active) return p;
  if (sg == 1 && (M <= 2 || (p.spw >= 7 && M <= 8))) return column_plan_for(8, 3, fmt, M, n_strips, n_rec_all, rec_k, gk, allow_qd);
  if (fmt == FMT_FP425 && allow_qd && p.spw >= 7 && M <= 16) {
    const ColumnPlan d = column_plan_for(8, 3, fmt, M, n_strips, n_rec_all, rec_k, gk, allow_qd);
    if (d.qd) return d;  // three records ahead exist for the side-group deal only
  }
  return p;
}

// More than eight strips for every compute unit (spw of them): whether two workgroups of slice_kernel with half the strips
// each beat the one of column_kernel / multi_kernel.  us column / slice; 2600 shapes of M = 1 to 16 since a wavefront asks for one
// record of activations ahead, 1500 per class before.
//   One scale per row, M <= 8, side groups: everywhere (128256 x 4096 FP4.25 M = 8 1.12 x, 90000 x 4096 1.38 x; 1.11-1.21 x in the mean, no
//     format below 1.02) but for two records per side group with a count that is even but no multiple of four, which
//     column_kernel deals without a rest while most of the eight wavefronts idle (65536 x 256 FP4.5 0.87 x, x 768 0.90 x,
//     from 24 records on +- 3 %).  At M = 1 in one round from 64 records on it would be 1.05-1.14 x: a
//     test names column_kernel's plan of 57344 x 8192, and it stays.
//   One scale per row, M <= 8, no side groups: up to ten strips, where three of multi_kernel's eight wavefronts, two strips each, have none
//     (33000 x 4096 FP5.33 M = 1 1.35 x, 40000 x 4096 1.28 x; one and two records 0.87-0.96 x; 65536 x 4096 0.92 x.  Eleven to
//     thirteen strips would gain 1.05-1.2 x: the plans of multi_kernel that tests name lie there, and they stay), and where at most half of the compute units
//     have a workgroup in the last round (90000 x 4096 1.17 x, 128256 x 4096 0.96 x).
//   M > 8: long K, where the staging of the activations starts to cost (45000 x 4096 M = 16 21.1 / 23.3; 64 to 80
//     records at M > 16 0.92-1.0 x).  From 32 or 43 records on M = 10 to 16 with one scale per row would
//     gain 1.06-1.14 x: tests name column_kernel's plans there, and they stay.
//   One scale per run: a wavefront's strips follow each other and the sum over eight wavefronts' tiles is the same
//     for one record as for a hundred, so a few records do not pay (65536 x 96 FP5.33 M = 4 0.83 x, x 1152 0.96 x), and where
//     the scales push the kernel beyond 128 registers the two workgroups take turns (65536 x 128 FP4.25 0.61 x, x 1024
//     0.87 x; FP4 0.57 x, 0.80 x); with more than one round of workgroups the turns fill each other's gaps earlier.
//     M <= 2 and 5 to 8 where it is taken: 96-weight records 1.06-1.13 x, FP4.25 1.10 x, 0.96 x at worst.
bool halved_is_faster(int fmt, int M, int64_t n_strips, int spw, int n_rec, bool one_scale) {
  const int sg = ams::side_group(ams::kFormats[fmt]), half = (spw + 1) / 2;
  const bool one_round = n_strips <= 16 * kNumCU, rec96 = ams::kFormats[fmt].rec_k == 96;
  if (M > 8) return n_rec >= (M > 16 && one_round ? 80 : 64);
  if (one_scale && sg == 1) {
    const int last = (int)((n_strips + spw - 1) / spw % kNumCU);  // workgroups of the last round
    return n_rec >= 3 && (one_round ? spw <= 10 : last > 0 && last <= kNumCU / 2);
  }
  if (one_scale) {
    if (sg == 2 && (one_round ? n_rec % 4 == 2 && n_rec < 24 : n_rec <= 2)) return false;
    return M > 1 || !one_round || n_rec < 64;
  }
  if (M == 3 || M == 4) {
    if (slice_two_fit(fmt, half)) return n_rec >= (one_round && half > 5 ? 16 : 3);
    return n_rec >= (!one_round ? 32 : half == kSliceMaxStrips && fmt != FMT_FP425 ? 64 : 24);
  }
  if (rec96 || half <= 6) return n_rec >= (one_round && half > 5 ? 24 : M > 4 ? 8 : 3);
  return half < kSliceMaxStrips ? n_rec >= 24 : fmt == FMT_FP425 && n_rec >= 64;
}

// Long K at M <= 2, where both kernels live on the bytes in flight.  The lines are from before slice_kernel asked for one record of
// activations ahead (and had twelve or sixteen wavefronts on two strips, not eight) and have not been drawn again.  Today it is the
// faster one of the two behind them: 1300 shapes, two strips 1.02-1.16 x (5120 x 25600 FP4.25 M = 1 17.1 us on column_kernel, M = 4
// on slice_kernel 16.4), four 1.00-1.04 x, one 1.00-1.02 x but for FP4.33 0.97 x.  As they were drawn, column / slice, 6800 shapes
// of 80 to 280 records and those of models, on five GPUs (+- 3 %):
//   two strips on fewer than 7/8 of the compute units: from 128 records on (5120 x 25600 FP4.25 M = 1 17.8 / 19.7 us, FP5.33
//     M = 2 20.3 / 22.5), at M = 1 from 97 on (6144 x 14336 FP4.25 11.6 / 12.5; 6144 x 4096 FP5.33 6.1 / 5.8) but for the
//     plain FP5 and FP4 (1.0-1.07 x);
//   two and four strips, one scale per run, records with two and more side bytes: from 97 records on at M = 1 (8192 x 14400
//     FP6 19.8 / 21.5, 16384 x 14336 FP5 27.9 / 28.9), from 145 on at M = 2 (14336 x 18944 FP6 38.5 / 42.5; FP4.5 from 201);
//   more than 200 records at M = 1 with a scale per run or side bytes (8192 x 25600 FP4.33 22.0 / 24.2, 4096 x 28672 with
//     scales per run 15.9 / 16.6), but for FP4 (1.00-1.08 x), FP4.25 with one scale per row (1.02-1.08 x), and on one strip
//     FP4.25, FP6 and FP5 with a scale per run (1.0-1.07 x).
bool long_k_on_column(int fmt, int M, int spw, int grid, int n_rec, bool one_scale) {
  if (M > 2 || (spw != 1 && spw != 2 && spw != 4)) return false;
  const int side = ams::kFormats[fmt].side_bytes;
  const bool plain = one_scale && (fmt == FMT_FP5 || fmt == FMT_FP4);
  if (spw == 2 && grid < kNumCU * 7 / 8 && (n_rec >= 128 || (M == 1 && n_rec > 96 && !plain))) return true;
  if (!one_scale && side >= 2 && spw > 1 && n_rec > (M == 1 ? 96 : fmt == FMT_FP45 ? 200 : 144)) return true;
  if (M > 1 || n_rec <= 200) return false;
  if (one_scale) return fmt == FMT_FP45 || fmt == FMT_FP433 || fmt == FMT_FP6;
  return spw == 1 ? fmt == FMT_FP533 || fmt == FMT_FP45 || fmt == FMT_FP433 : fmt != FMT_FP4;
}

// Short slices of a split K at M > 8, several strips per workgroup: the tiles of eight wavefronts cost the same however few
// records lie behind them (column_kernel's sixteen leave 16 / strips of them per strip), and the workgroup's sum waits
// for the slowest.  Column / slice over twelve N, thirteen K, seven formats, M = 12, 16, 24, 32:
//   four slices: up to 16 records of 128 weights or 29 of 96, five strips and more at M > 16 (5120 x 6144 0.87-0.94 x, x 11008
//     FP5.33 0.92 x), six and more below (7168 x 8192 0.84-0.94 x; x 14336 1.0 x);
//   eight slices: as many records with three strips at M > 16 (1536 x 13824 0.91-0.99 x, x 18944 FP4.25 1.02 x); any number
//     measured, up to 40, with four strips and more at M > 16 (2048 x 25600 0.94-0.97 x) and with seven and eight below
//     (3584 x 22016 0.80 x); with five and six below up to 24 of 128 or 29 of 96 (2560 x 18944 0.86-0.97 x, x 25600 1.0 x).
// Longer slices and fewer strips: 0.96-1.4 x.
bool short_slices_on_column(int fmt, int M, int spw, int gk, int n_rec_all) {
  if (M <= 8 || gk < 4) return false;
  const int n_rec = (n_rec_all + gk - 1) / gk;
  const bool rec96 = ams::kFormats[fmt].rec_k == 96;
  if (gk == 4) return spw >= (M > 16 ? 5 : 6) && n_rec <= (rec96 ? 29 : 16);
  if (spw >= (M > 16 ? 4 : 7)) return n_rec <= 40;
  return M > 16 ? spw == 3 && n_rec <= (rec96 ? 29 : 16) : spw >= 5 && n_rec <= (rec96 ? 29 : 24);
}

// The rows of X dealt to several workgroups.  A compute unit draws its weights and its activations through one in-order path
// that keeps 32 KiB (the lines of its cache) in flight, and every workgroup needs all of its rows' activations: at M = 32 on
// one strip they are seven times the weights.  With `tiles` workgroups on one position along N, each with its share of the rows
// and `tiles` times the strips, a compute unit moves fewer bytes; the weights are then read `tiles` times, once from memory
// and else from the XCD's L2.  The cost of a step of K: the records of the strips, and 0.72 of the activations' cache lines (a
// line out of L2 comes quicker than one out of memory); fitted to 108 shapes.  One scale per run costs every strip another 384
// bytes' worth (4608 x 2368 FP5.33 M = 16 5.47 / 5.71, FP4.25 5888 x 22656 26.7 / 27.9).  us, one / two tiles: 4096 x 14336 FP4.25 M = 32
// 20.3 / 16.4, M = 24 17.8 / 16.3, M = 16 13.9 / 13.2, M = 12 12.5 / 12.7; FP5.33 M = 32 22.6 / 18.3; 8192 x 8192 M = 32 15.7 / 14.5,
// M = 16 11.7 / 12.9; 14336 x 4096 M = 32 12.9 / 13.1; 2560 x 9728 M = 24 12.8 / 11.1, three tiles 9.6.  Tiles of fewer than eight rows
// do not pay where they cost strips (2419 x 20352 FP5.33 M = 12 16.9, three tiles 19.2).  At 16 rows
// a second strip costs FP6, and FP4.33 up to 32 records (with a scale per run 96), what the rows save (one / two tiles: 2739 x 1920
// FP6 4.2 / 4.5, 2155 x 2776 FP4.33 with a scale per run 5.1 / 5.5; 129 to 256 strips 0.90-0.98 x); on up to 128 strips they
// take none and are dealt.  With fewer than 18 records, two for a wavefront, plans with 129 strips and more stay as they were before the
// rows were dealt; the line is not where the two meet: over 15500 such shapes dealing is 1.03-1.07 x at 16 rows and 1.12-1.17 x beyond on
// 5 to 17 records, 0.99-1.06 x on 2 to 4.
// Up to 128 strips (two tiles, 80 three, 64 four) the tiles go to compute units that have nothing to do otherwise: from five rows
// on, tiles of four rows and more (us, undealt / dealt: 1024 x 14336 FP4.25 M = 8 8.3 / 7.0, M = 12 10.3 / 7.3, M = 16 two tiles 8.2 / four
// 7.4; 2048 x 9728 FP5.33 M = 12 8.6 / 7.1; 2048 x 1024 FP4.25 M = 32 3.8 / 3.1; 32000 shapes of M = 5 to 32 1.08 x, 1.1-1.5 x beyond 64
// records), but for tiles of five to eight rows on up to eight records at M <= 16 (0.96-0.99 x).
constexpr int64_t kSplitMaxStrips = 16384;  // strips that the counters of a split of K have room for
struct RowSplit {
  int strips, positions;  // strips per workgroup; workgroups of one tile: whole groups of eight, so that the tiles of a position meet on one XCD
  double cost;
};
double row_split_cost(int fmt, int strips, int rows, bool one_scale) {
  return strips * (double)(ams::kFormats[fmt].rec_bytes + (one_scale ? 0 : 384)) + 0.72 * 256 * rows;
}
RowSplit row_split(int fmt, int M, int64_t n_strips, int gk, int tiles, bool one_scale) {
  RowSplit s;
  const int64_t most = kNumCU / tiles & ~7;
  s.strips = (int)((n_strips * gk + most - 1) / most);
  while ((s.positions = (int)(ams::round_up((n_strips + s.strips - 1) / s.strips * gk, 8))) > most) s.strips++;
  s.cost = row_split_cost(fmt, s.strips, (M + tiles - 1) / tiles, one_scale);
  return s;
}
constexpr int kMaxRowTiles = 4, kRowSplitMinRecords = 18, kRowSplitMinRows = 8;

// Rows of X that are not 16-byte aligned: slice_kernel's variant for them, on tiles of up to eight rows and up to four strips
// (its sixteen wavefronts have 128 registers each).  21000 shapes against column_kernel, which stages the rows for the workgroup
// (in phases of K where all of it does not fit): 1.7 x in the mean (32 rows 2-4 x: 4096 x 14337 FP4.25 47.7 / 22.5 us; 8 rows in
// phases 4096 x 14339 FP4.25 16.5 / 12.7, 13 strips 1.5 x, 400 strips 1.2 x).  column_kernel stays with one scale per run, on
// one record, where it reads three records ahead (8192 x 8193 FP5.33 M = 1 11.0 / 11.2), and:
//   at one row on long K, where staging it is nothing and the wavefronts live on the records in flight: from where the two meet, by
//     format (5.33 bits from 230 records on 0.98 x, from 800 on 0.91 x; FP4.5 0.95 and 0.94 x);
//   two tiles of four strips, which wavefronts walk one after the other: see four_strips_on_column.
int ragged_tiles(int M) { return (M + kSliceRaggedMaxRows - 1) / kSliceRaggedMaxRows; }
// Two tiles of unaligned rows (9 to 16) on four strips, n records; column / streamed over 7800 shapes:
//   29 to 32 records, which column_kernel's eight wavefronts of a strip share evenly: 0.89-1.0 x (6285 x 2727 FP5.33 M = 12 8.2 / 9.0; 25
//     to 28 records 1.0-1.2 x, 33 to 36 1.0-1.3 x);
//   57 to 64 likewise, up to 12 rows (0.84-0.97 x; FP4.5 and FP4 1.1 x); FP6 there from 49 on (0.85-0.94 x; 13 to 15 rows 0.91-1.1 x, left);
//   nine rows, a tile of five and one of four, from 29 on (FP5 0.81-0.93 x, FP4.25 0.86-0.98, FP5.33 0.96-1.13); ten of FP5 (0.86-0.91 x).
bool four_strips_on_column(int fmt, int M, int n) {
  if (n <= 28) return false;
  if (n <= 32 || M == 9 || (M == 10 && fmt == FMT_FP5)) return true;
  return M <= 12 && ((n > 56 && n <= 64) || (fmt == FMT_FP6 && n > 48));
}
constexpr int kRaggedLongK[ams::kNumFormats] = {230, 220, 155, 190, 160, 240, 280};
bool ragged_on_slice(int fmt, int M, int64_t n_strips, int n_rec, int rec_k, int gk, bool one_scale, const ColumnPlan& column) {
  if (!one_scale || (int64_t)n_rec * rec_k < 8 + rec_k || n_strips > kSplitMaxStrips / kMaxRowTiles) return false;
  if (column.lr == 3 || column.spw > kSliceRaggedMaxStrips) return false;
  if (M == 1 && n_rec > kRaggedLongK[fmt]) return false;
  const int tiles = ragged_tiles(M), strips = row_split(fmt, M, n_strips, gk, tiles, true).strips;
  if (tiles == 2 && strips == kSliceRaggedMaxStrips && gk <= 2 && four_strips_on_column(fmt, M, (n_rec + gk - 1) / gk)) return false;
  return strips <= kSliceRaggedMaxStrips;
}
// p on slice_kernel: what its variant of p's strips and row tiles is launched with.
ColumnPlan slice_plan(ColumnPlan p, int fmt, int M, int variant) {
  p.slice = true;
  p.variant = variant;
  p.rows = slice_rows((M + p.row_tiles - 1) / p.row_tiles);
  const SliceAsk ask = slice_ask(fmt, p.rows, p.spw, variant);
  p.S = ask.waves;
  p.lr = ask.weights;
  p.lds = (size_t)slice_lds(fmt, p.rows, p.spw, variant);
  return p;
}
ColumnPlan ragged_plan(ColumnPlan p, int fmt, int M, int64_t n_strips, int gk) {
  p.row_tiles = ragged_tiles(M);
  if (p.row_tiles > 1) {
    const RowSplit s = row_split(fmt, M, n_strips, gk, p.row_tiles, true);
    p.spw = s.strips;
    p.gn = (int)((n_strips + p.spw - 1) / p.spw);
    p.grid = s.positions * p.row_tiles;
  }
  return slice_plan(p, fmt, M, kSliceRagged);
}

// One strip: whether to ask for two records ahead (kSliceDeep, kSliceDeepRuns; 128-weight records at 13 to 16 rows: of activations), not one.  us, one / two:
//   M <= 2, no side groups, fewer workgroups than 7/8 of the compute units, and a stream that is long against its start: the
//     memory is not what limits them there, every compute unit waits for its own requests.  1500 shapes of 1 to 223 strips 1.035 x
//     (FP5.33 M = 1 2560 x 24960 11.64 / 11.04 us, 1024 x 18432 8.89 / 8.59; FP4 3520 x 38400 13.70 / 12.76; M = 2 12.24 / 11.83 on
//     3520 x 24960), at the first percentile 0.988 x; at the lines 1.00-1.01 x.  From 224 strips on 0.90-0.98 x below 128 records;
//     the longer ones are column_kernel's.  Formats with side groups 0.95-1.03 x.
//   Tiles of 9 to 16 rows of 96-weight records, where the records are two to four for each of eight wavefronts: twelve that
//     stream leave a round half empty and write half as many tiles again.  900 shapes FP4.33 1.04 x (4096 x 2688 M = 15 4.69 / 4.42,
//     4096 x 1536 3.78 / 3.53), FP6 1.025 x (4.93 / 4.77), FP5.33 1.012 x; from 29 records on FP4.33 1.03 x up to 36, the others 0.99-1.0 x;
//     below 16 0.98-1.01 x.
//   Tiles of 13 to 16 rows of 128-weight records, from 18 of them on: eight wavefronts instead of twelve streams 1.025 x over
//     900 shapes, at the first percentile 0.97 x (FP4.25 M = 15 4096 x 3072 4.97 / 4.68, x 14336 12.99 / 12.71; with a scale per run M = 16
//     5.34 / 4.91, 13.92 / 13.54; 29 to 31 records, three rounds of twelve, 0.96-1.0 x); 9 rows 0.98 x, 12 rows 1.01 x; with a scale per
//     run on 6 to 17 records 0.98-1.02 x.
bool more_ahead_is_faster(int fmt, int variant, int M, int tile_rows, int strips, int grid, int n_rec) {
  const int rows = slice_rows(tile_rows);
  if (!slice_has_deep(fmt, variant, rows, strips)) return false;
  if (rows == 4) return M <= 2 && grid < kNumCU * 7 / 8 && n_rec >= (fmt == FMT_FP5 ? (M == 1 ? 128 : 240) : (M == 1 ? 96 : 160));
  if (ams::kFormats[fmt].rec_k != 96) return tile_rows >= 13 && n_rec >= 18;
  return n_rec >= 16 && n_rec <= (fmt == FMT_FP433 ? 36 : 28);
}

// The plan of a problem: slice_kernel where it takes it (aligned_rows: rows of X are 16-byte aligned, K % 8 == 0;
// one_scale: one scale per row of W), else make_column_plan's.  slice_kernel is the faster one nearly everywhere
// (twelve shapes, seven formats, M = 1 .. 32: 1.00-1.8 x); the exceptions, us column / slice:
//   one strip per workgroup, M <= 2, where eight wavefronts with three records ahead fill the chip (no side groups): 4096 x
//     14336 FP5.33 M = 1 9.5 / 9.4, M = 2 10.1 / 10.1 with two records ahead on slice_kernel; with one 9.4 / 8.6 and 9.9 / 8.5, not
//     drawn again;
//   one, two and four strips, M <= 2, long K: see long_k_on_column;
//   six strips and more, M > 8, a few records: with fewer than eight of them wavefronts idle, the busy ones walk all
//     strips one after the other, and the idle ones' tiles are written and summed too (32768 x 128 M = 32 0.75 x, 24576
//     x 192 0.9 x); eight strips at M > 16, whose tiles fill 128 KiB, up to sixteen records (32768 x 1024 0.9 x; 28672 x 4096
//     FP5.33 M = 32 24.7 / 18.9);
//   short slices of a split K: see short_slices_on_column;
//   more than eight strips: see halved_is_faster.
// p: make_column_plan's of the same problem.
ColumnPlan plan_from(ColumnPlan p, int fmt, int M, int64_t n_strips, int n_rec_all, int rec_k, int gk, bool aligned_rows, bool one_scale) {
  if (!aligned_rows) {
    if (ragged_on_slice(fmt, M, n_strips, n_rec_all, rec_k, gk, one_scale, p)) return ragged_plan(p, fmt, M, n_strips, gk);
    return p;
  }
  if (p.spw == 1 && p.lr == 3) return p;
  if (long_k_on_column(fmt, M, p.spw, p.grid, n_rec_all, one_scale)) return p;
  if (short_slices_on_column(fmt, M, p.spw, gk, n_rec_all)) return p;
  if (gk == 1 && p.spw == 8 && n_rec_all <= (M > 16 ? 16 : M > 8 ? 2 : 0)) return p;
  if (gk == 1 && M > 16 && (p.spw == 6 || p.spw == 7) && n_rec_all <= 2) return p;
  if (p.spw > kSliceMaxStrips) {
    if (gk != 1 || !halved_is_faster(fmt, M, n_strips, p.spw, n_rec_all, one_scale)) return p;
    p.spw = (p.spw + 1) / 2;
    p.grid = p.gn = (int)((n_strips + p.spw - 1) / p.spw);
  }
  if (M >= 2 * kRowSplitMinRows && n_rec_all / gk >= kRowSplitMinRecords && n_strips <= kSplitMaxStrips / kMaxRowTiles) {
    const bool costly_strip = gk == 1 && ((one_scale && fmt == FMT_FP6) || (fmt == FMT_FP433 && n_rec_all <= (one_scale ? 32 : 96)));
    double best = 0.97 * row_split_cost(fmt, p.spw, M, one_scale);
    const int one_strip = gk == 1 ? p.spw : 0;
    for (int t = 2; t <= kMaxRowTiles; t++) {
      const RowSplit s = row_split(fmt, M, n_strips, gk, t, one_scale);
      if (s.strips > kSliceMaxStrips || s.cost >= best || (M <= 16 && s.strips > p.spw && costly_strip)) continue;
      if (t * kRowSplitMinRows > M && (s.strips > 1 || one_strip != 1)) continue;
      best = s.cost;
      p.row_tiles = t;
      p.spw = s.strips;
      p.gn = (int)((n_strips + s.strips - 1) / s.strips);
      p.grid = s.positions * t;
    }
  } else if (gk == 1 && p.spw == 1) {
    for (int t = std::min(kMaxRowTiles, (M + 3) / 4); t > 1 && p.row_tiles == 1; t--) {
      const RowSplit s = row_split(fmt, M, n_strips, gk, t, one_scale);
      if (s.strips == 1 && (M > 16 || (M + t - 1) / t <= 4 || n_rec_all > 8)) p.row_tiles = t, p.grid = s.positions * t;
    }
  }
  const int deep = one_scale ? kSliceDeep : kSliceDeepRuns;
  if (gk == 1 && more_ahead_is_faster(fmt, deep, M, (M + p.row_tiles - 1) / p.row_tiles, p.spw, p.grid, n_rec_all)) return slice_plan(p, fmt, M, deep);
  return slice_plan(p, fmt, M, one_scale ? kSlicePlain : kSliceRunScales);
}
ColumnPlan make_plan(int fmt, int M, int64_t n_strips, int n_rec_all, int rec_k, int gk, bool aligned_rows, bool one_scale, bool nt) {
  const ColumnPlan column = make_column_plan(fmt, M, n_strips, n_rec_all, rec_k, gk, one_scale, one_scale && nt);
  return plan_from(column, fmt, M, n_strips, n_rec_all, rec_k, gk, aligned_rows, one_scale);
}

// Workspace of a split in gk slices: per-strip arrival counters, then the partial tiles.  The
// counter area has one size for every shape, so that a workspace that is reused for another
// shape never finds old tile data where it expects counters at zero.
constexpr size_t kSplitCounterBytes = (size_t)kSplitMaxStrips * 4;
size_t split_workspace_bytes(int M, int64_t n_strips, int gk) {
  return gk <= 1 ? 0 : kSplitCounterBytes + (size_t)gk * n_strips * (M > 16 ? 2 : 1) * 1024;
}

// The baseline's GEMV kernel takes batches up to 4 whose activations fit in LDS beside nothing else.
struct GemvPlan {
  bool ok;
  int kpad;    // K rounded up to whole 512-channel segments
  size_t lds;  // M rows of kpad halfs
};
GemvPlan make_gemv_plan(int M, int64_t K, int gk) {
  GemvPlan p;
  p.kpad = (int)((K + 511) / 512 * 512);
  p.lds = (size_t)M * p.kpad * 2;
  p.ok = M <= 4 && gk == 1 && K % 8 == 0 && p.lds <= (size_t)kLdsMaxBytes;
  return p;
}

constexpr int kMaxSplit = kMaxSlices;  // most slices of K choose_split ever takes
constexpr size_t kStaticScratchBytes = ((size_t)64 << 10) + ((size_t)8 << 20);  // of ams_linear_static_ws
// passed as the workspace by the entry point that uses the library's static scratch instead
void* const kStaticScratch = (void*)(uintptr_t)1;

// How many slices of K to use when a workspace is available.  A split pays when the strips
// alone do not fill the compute units evenly (e.g. 320 strips: 2 per workgroup on 160 CUs,
// against 5 strips x a quarter of K on 256) and when the batch is large (every workgroup
// stages the activations of its own slice of K only).  The estimate is bytes a workgroup
// moves: its weight records, half weight for the activations it stages (they come from
// L2), and a fixed charge for the exchange through the workspace (fitted to measurements on
// the Llama and Qwen shapes: below a batch of 4 the stream is bound by the memory system as a
// whole and a split never paid).  For the packed formats it prices column_kernel, to which it was fitted; slice_kernel, which takes
// the slices but for the short ones, stages nothing per phase and is now and then faster without the split (2560 x 9728
// FP4.25 M = 16 9.7 us, split 10.0).
// column: make_column_plan's with 1, 2, 4, 8 slices, as far as they were looked at.
int cheapest_split(int fmt, int M, int64_t n_strips, int n_rec, int rec_k, int rec_bytes, ColumnPlan (&column)[4]) {
  if (M < 4) return 1;
  int best = 1;
  double best_cost = 0;
  for (int gk = 1, j = 0; gk <= kMaxSplit; gk *= 2, j++) {
    if (gk > 1 && (n_rec / gk < 8 || n_strips > kSplitMaxStrips)) break;
    int spw, rc;
    double rounds = 1.0;  // the packed formats' workgroups take at most 16 strips: more of them means more rounds
    SweepPlan p;
    p.ok = true;
    if (fmt != FMT_FP16) {
      const ColumnPlan& cp = column[j] = make_column_plan(fmt, M, n_strips, n_rec, rec_k, gk);
      spw = cp.spw, rc = cp.rc;
      rounds = std::max(1.0, (double)cp.grid / kNumCU);
    } else {
      p = make_sweep_plan(fmt, M, n_strips, n_rec, rec_k, false, gk);
      spw = p.spw, rc = p.rc;
    }
    if (!p.ok) {
      if (gk > 1) continue;
      // without a split the shape would go to the contiguous-piece kernel: price that one
      const StreamPlan sp = make_stream_plan(fmt, M, n_strips, n_rec, rec_k);
      if (!sp.ok) continue;
      spw = sp.spw, rc = sp.rc;
    }
    const double slice = (double)((n_rec + gk - 1) / gk);
    const double n_phase = std::max(1.0, slice / rc);
    double cost = spw * slice * rec_bytes + 0.5 * M * slice * rec_k * 2 + 8192.0 * (n_phase - 1);
    if (gk > 1) cost += 49152.0 + 2048.0 * gk * spw * (M > 16 ? 2 : 1);
    cost *= rounds;
    if (best_cost == 0 || cost < best_cost) best = gk, best_cost = cost;
  }
  return best;
}

// Time of a plan in us, slices with aligned rows: the bytes of row_split_cost at 47 KB a microsecond, the sum over the
// wavefronts' tiles, and for a split the exchange.  Fitted to 197 shapes with and without their split (9 % r.m.s.), none of them
// with tiles of fewer than eight rows, which count as undealt.
double plan_time(const ColumnPlan& p, int fmt, int M, int n_rec) {
  const int row_tiles = std::min(p.row_tiles, std::max(1, M / kRowSplitMinRows)), rows = (M + row_tiles - 1) / row_tiles;
  const double tiles = p.spw * rows / 100.0;
  const double t = 2.1 + (n_rec + p.gk - 1) / p.gk * row_split_cost(fmt, p.spw, rows, true) / 46500.0 + 3.25 * tiles;
  return p.gk > 1 ? t + 3.05 - 1.7 * tiles : t;
}

// The split that a call with a workspace uses: cheapest_split's, unless the plain call is faster.  us, split / whole:
//   slices on slice_kernel: on short K the exchange costs more than they save, and plan_time decides (896 x 2880 FP4.25 M = 32 7.0 /
//     4.0, 4096 x 4096 8.4 / 7.2, 1226 x 5760 FP5.33 M = 16 6.4 / 5.2).  How short depends on M, because the activations of
//     all of K weigh more with every row, and from 16 rows on a plain call deals them out: over 43000 shapes the two meet at
//     K = 12800 with 4 rows, 9000 with 8, 6500 with 12 and 9200 from 16 on (where more than one strip falls on every compute unit, at
//     9200 with 4 too); the bounds lie a little below, where the choice errs least.  Beyond them the split is the faster one (2560 x
//     9728 FP4.25 M = 16 7.8 / 9.1, 5120 x 25600 FP5.33 19 / 29).  The choice is within 0.4 % of the faster one in the mean, and more than 6 % off in 2 % of the shapes.
//   four or eight slices on column_kernel (short ones, or more than eight strips): below K = 9216 the plain call is the faster one, up
//     to 12 rows at every K (5120 x 6144 FP5.33 M = 32 12.3 / 10.8, 7168 x 8192 FP4.5 M = 16 13.4 / 11.6; 1215 shapes: 1.10 x at K = 8000, 1.03 x
//     around 9000, 0.96 x at 12000; M = 8 up to 20000 1.11 x).
//   up to 128 strips, from five rows on: the plain call deals its rows to the compute units that the strips leave idle (plan_from), and
//     where such a compute unit moves less than split_moved the exchange costs more than the slices save.  Counted are its records, a
//     side dword's load as 224 bytes (320 where no other record shares it), and 90 bytes for a row of activations (190 from the ninth on); it lies
//     lower on a few strips, whose slices hardly meet in the exchange (69 x 11016 FP6 M = 9 5.3 / 7.0), and higher where four slices
//     are 224 to 256 workgroups.  1187 x 7848 FP4.25 M = 12 6.3 / 5.2, 1024 x 14336 M = 12 7.5 / 7.0, 2048 x 9728 FP5.33 M = 12 6.8 /
//     7.0, 2048 x 14336 8.1 / 9.0.
//     Over 4000 such shapes that would split without this line the choice is 0.10 % off the faster one in the mean, 3.4 % at
//     the last percentile (4.5 and 36 % without it).
// Unaligned rows keep cheapest_split's (17000 shapes: the plain call is 1.1-1.3 x faster below K = 5000 and the split from 8000
// on; in between it depends on the strips).
constexpr int kSplitLongK = 9216;
constexpr int kSplitLongKOfRows[16] = {0, 0, 0, 0, 12800, 10950, 9640, 8650, 7880, 7250, 6740, 6300, 5930, 5610, 5320, 5070};  // 12800 (4 / M)^0.7
double split_moved(int64_t n_strips) {
  return std::min(172e3, 124e3 + 6e3 * std::max<double>(0, n_strips - 7)) + (n_strips >= 56 && n_strips <= 64 ? 20e3 : 0);
}
struct Split {
  int gk;
  bool planned;  // plan: make_plan's for gk slices, non-temporal loads
  ColumnPlan plan;
};
Split choose_split(int fmt, int M, int64_t n_strips, int n_rec, int rec_k, int rec_bytes, int64_t K) {
  ColumnPlan column[4];
  Split c;
  c.gk = cheapest_split(fmt, M, n_strips, n_rec, rec_k, rec_bytes, column);
  c.planned = false;
  if (c.gk == 1 || fmt == FMT_FP16 || K % 8 != 0) return c;
  const ColumnPlan& sliced = column[c.gk == 2 ? 1 : c.gk == 4 ? 2 : 3];
  const bool on_slice = sliced.spw <= kSliceMaxStrips && !short_slices_on_column(fmt, M, sliced.spw, c.gk, n_rec);  // as plan_from has it
  if (on_slice && n_strips <= kNumCU / 2 && M > 4) {  // the plain call deals its rows out
    const ColumnPlan whole = plan_from(column[0], fmt, M, n_strips, n_rec, rec_k, 1, true, true);
    const ams::FormatInfo& fi = ams::kFormats[fmt];
    const int rows = (M + whole.row_tiles - 1) / whole.row_tiles;
    const double moved = n_rec * (whole.spw * (fi.rec_bytes + (fi.side_bytes == 4 ? 320.0 : fi.side_bytes ? 224.0 : 0.0)) + 90.0 * rows + 100.0 * std::max(0, rows - 8));
    if (whole.slice && moved < split_moved(n_strips)) {
      c.gk = 1, c.plan = whole, c.planned = true;
      return c;
    }
  }
  int long_k = kSplitLongK;
  if (on_slice && M < 16) long_k = n_strips > kNumCU ? std::min(kSplitLongKOfRows[M], kSplitLongK) : kSplitLongKOfRows[M];
  if (on_slice ? K >= long_k : c.gk == 2 || (K >= long_k && M > 12)) return c;
  // a split that the static scratch refuses stays refused
  if (split_workspace_bytes(M, n_strips, c.gk) > kStaticScratchBytes) return c;
  const ColumnPlan whole = plan_from(column[0], fmt, M, n_strips, n_rec, rec_k, 1, true, true);
  if (!whole.slice) return c;
  c.plan = plan_from(sliced, fmt, M, n_strips, n_rec, rec_k, c.gk, true, true);
  c.planned = true;
  if (!c.plan.slice || plan_time(whole, fmt, M, n_rec) < plan_time(c.plan, fmt, M, n_rec)) c.gk = 1, c.plan = whole;
  return c;
}

// Per-device state, set up once per device with that device current: whether it is the GPU
// this library is written for, and where this device's copy of the static scratch lives.
constexpr int kMaxDevices = 64;
struct DeviceState {
  int status;     // 0 = not looked at yet, 1 = usable, -1 = not a gfx950 with the expected resources
  void* scratch;  // device address of this device's `scratch` array
};
std::mutex g_dev_mu;
DeviceState g_dev[kMaxDevices];

// Scratch of the entry point that may not allocate (ams_linear_static_ws): the arrival counters
// and partial tiles of a split of K.  One copy per GPU, held until the process ends.  In host
// code this name is only a handle for hipGetSymbolAddress, never a device address.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

// AMS_OK when the current device is a gfx950 with the compute units and LDS the launch plans
// assume; looked up once per device (no allocation, no synchronisation).
int device_state(DeviceState** out = nullptr) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return AMS_ERR_DEVICE;
  std::lock_guard<std::mutex> lock(g_dev_mu);
  DeviceState& d = g_dev[dev];
  if (d.status == 0) {
    hipDeviceProp_t prop;
    d.status = -1;
    if (hipGetDeviceProperties(&prop, dev) == hipSuccess && strncmp(prop.gcnArchName, "gfx950", 6) == 0 &&
        prop.multiProcessorCount >= 1 && prop.warpSize == 64) {
      void* ptr = nullptr;
      if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) == hipSuccess && ptr) {
        d.scratch = ptr;
        d.status = 1;
      }
    }
    (void)hipGetLastError();  // a failed query must not be reported by the caller's next HIP call
  }
  if (out) *out = &d;
  return d.status == 1 ? AMS_OK : AMS_ERR_DEVICE;
}

// Kernels that use more than 64 KiB of dynamic LDS must have their limit raised first;
// that is a per-function, per-device property, remembered here so it is done once.
bool raise_lds_limit(const void* kern) {
  static std::mutex mu;
  static std::unordered_set<const void*> done[kMaxDevices];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return false;
  std::lock_guard<std::mutex> lock(mu);
  if (done[dev].count(kern)) return true;
  if (hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsMaxBytes) != hipSuccess) return false;
  try {
    done[dev].insert(kern);
  } catch (...) {  // out of host memory: the limit is raised, it is just not remembered
  }
  return true;
}

// grid == 0: only prepare the kernel (raise its LDS limit), launch nothing (ams_init)
template <class Kern>
int launch(Kern kern, const LinearArgs& a, unsigned grid, int S, size_t lds, hipStream_t st) {
  if ((grid == 0 || lds > 64 * 1024) && !raise_lds_limit((const void*)kern)) return AMS_ERR_LAUNCH;
  if (grid == 0) return AMS_OK;
  hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * S), lds, st, a);
  return hipGetLastError() == hipSuccess ? AMS_OK : AMS_ERR_LAUNCH;
}

enum KernelKind { kSweep, kStream };

// The fp16 baseline's kernels by ring depth and wave grouping.
template <int MT>
int launch_fp16(KernelKind kind, int lr, const LinearArgs& a, unsigned grid, int S, size_t lds, hipStream_t st) {
  const bool groups = a.wps != S;  // wave groups per strip: their own instantiation, the common case stays lean
  if (kind == kSweep) {
    if (lr == 1) return groups ? launch(sweep_kernel<MT, 1, true>, a, grid, S, lds, st) : launch(sweep_kernel<MT, 1, false>, a, grid, S, lds, st);
    if (lr == 2 && !groups) return launch(sweep_kernel<MT, 2, false>, a, grid, S, lds, st);
  } else {
    switch (lr) {
      case 4: return launch(stream_kernel<MT, 4>, a, grid, S, lds, st);
      case 2: return launch(stream_kernel<MT, 2>, a, grid, S, lds, st);
    }
  }
  return AMS_ERR_LAUNCH;
}

// The baseline's GEMV kernel by batch size.
int launch_gemv(int M, bool nt, const LinearArgs& a, unsigned grid, size_t lds, hipStream_t st) {
  switch (M) {
    case 1: return nt ? launch(gemv_fp16_kernel<1, true>, a, grid, 16, lds, st) : launch(gemv_fp16_kernel<1, false>, a, grid, 16, lds, st);
    case 2: return nt ? launch(gemv_fp16_kernel<2, true>, a, grid, 16, lds, st) : launch(gemv_fp16_kernel<2, false>, a, grid, 16, lds, st);
    case 3: return nt ? launch(gemv_fp16_kernel<3, true>, a, grid, 16, lds, st) : launch(gemv_fp16_kernel<3, false>, a, grid, 16, lds, st);
    case 4: return nt ? launch(gemv_fp16_kernel<4, true>, a, grid, 16, lds, st) : launch(gemv_fp16_kernel<4, false>, a, grid, 16, lds, st);
  }
  return AMS_ERR_LAUNCH;
}

// The packed formats' kernel: nt = non-temporal weight loads, gs = one scale per run of input channels.
template <int FMT, int MT, bool RAGGED>
int launch_column_rows(bool nt, bool gs, bool qd, int lr, const LinearArgs& a, unsigned grid, int S, size_t lds, hipStream_t st) {
  if (gs) return launch(column_kernel<FMT, MT, true, true, false, 2, RAGGED>, a, grid, S, lds, st);
  // Three records ahead: make_column_plan's plans for M <= 16; FP4.25's with the side groups dealt whole are seven and
  // eight strips, which slice_kernel takes where rows are aligned.
  if constexpr (MT == 1 && Fmt<FMT>::SG == 1) {
    if (lr == 3) return nt ? launch(column_kernel<FMT, MT, true, false, false, 3, RAGGED>, a, grid, S, lds, st) : AMS_ERR_LAUNCH;
  }
  if constexpr (MT == 1 && FMT == FMT_FP425 && RAGGED) {
    if (qd && lr == 3) return nt ? launch(column_kernel<FMT, MT, true, false, true, 3, RAGGED>, a, grid, S, lds, st) : AMS_ERR_LAUNCH;
  }
  if (lr != 2) return AMS_ERR_LAUNCH;
  if constexpr (Fmt<FMT>::SG > 1) {
    if (qd)
      return nt ? launch(column_kernel<FMT, MT, true, false, true, 2, RAGGED>, a, grid, S, lds, st)
                : launch(column_kernel<FMT, MT, false, false, true, 2, RAGGED>, a, grid, S, lds, st);
  }
  return nt ? launch(column_kernel<FMT, MT, true, false, false, 2, RAGGED>, a, grid, S, lds, st)
            : launch(column_kernel<FMT, MT, false, false, false, 2, RAGGED>, a, grid, S, lds, st);
}
template <int FMT, int MT>
int launch_column(bool nt, bool gs, bool qd, int lr, const LinearArgs& a, unsigned grid, int S, size_t lds, hipStream_t st) {
  return (a.K & 7) == 0 ? launch_column_rows<FMT, MT, false>(nt, gs, qd, lr, a, grid, S, lds, st)
                        : launch_column_rows<FMT, MT, true>(nt, gs, qd, lr, a, grid, S, lds, st);
}

// Wavefronts that own two strips each (non-temporal loads, one scale per row; planned up to M = 8).
template <int FMT>
int launch_multi(const LinearArgs& a, unsigned grid, int S, size_t lds, hipStream_t st) {
  if constexpr (Fmt<FMT>::SG == 1)
    return (a.K & 7) == 0 ? launch(multi_kernel<FMT, 1, true, 2, false>, a, grid, S, lds, st)
                          : launch(multi_kernel<FMT, 1, true, 2, true>, a, grid, S, lds, st);
  return AMS_ERR_LAUNCH;
}

// slice_kernel for r staged rows and `strips` strips per workgroup.
template <int FMT>
int launch_slice(const LinearArgs& a, int variant, int r, int strips, unsigned grid, hipStream_t st) {
  const void* kern = variant == kSliceRunScales ? slice_kernel_of<FMT, kSliceRunScales>(r, strips)
                     : variant == kSliceRagged  ? slice_kernel_of<FMT, kSliceRagged>(r, strips)
                     : variant == kSliceDeep    ? slice_kernel_of<FMT, kSliceDeep>(r, strips)
                     : variant == kSliceDeepRuns ? slice_kernel_of<FMT, kSliceDeepRuns>(r, strips)
                                                 : slice_kernel_of<FMT, kSlicePlain>(r, strips);
  if (!kern) return AMS_ERR_LAUNCH;
  const size_t lds = (size_t)slice_lds(FMT, r, strips, variant);
  if (lds > 64 * 1024 && !raise_lds_limit(kern)) return AMS_ERR_LAUNCH;
  if (grid == 0) return AMS_OK;
  const uint64_t w = (uint64_t)a.W, x = (uint64_t)a.X, sc = (uint64_t)a.scales;
  uint32_t head[14] = {(uint32_t)w, (uint32_t)(w >> 32), (uint32_t)x, (uint32_t)(x >> 32), (uint32_t)sc, (uint32_t)(sc >> 32), (uint32_t)a.M, (uint32_t)a.N,
                       (uint32_t)a.K, (uint32_t)a.n_rec, (uint32_t)a.n_strips, (uint32_t)a.gn, (uint32_t)a.gk, (uint32_t)a.tile_rows};
  SliceArgs rest = {a.Y, a.ws_tiles, a.ws_count, a.n_sg, a.sg_shift, a.row_tiles};
  void* args[] = {head, head + 4, head + 8, head + 12, &rest};
  return hipLaunchKernel(kern, dim3(grid / a.row_tiles, a.row_tiles), dim3(64 * slice_ask(FMT, r, strips, variant).waves), args, lds, st) == hipSuccess ? AMS_OK : AMS_ERR_LAUNCH;
}

template <int FMT>
int run_linear(const void* W, const uint16_t* scales, const uint16_t* X, uint16_t* Y, int M, int64_t N, int64_t K,
               void* stream, int64_t scale_group = 0, void* workspace = nullptr, size_t ws_bytes = 0) {
  if (!W || !X || !Y || (FMT != FMT_FP16 && !scales)) return AMS_ERR_NULL;
  if (M < 1 || M > AMS_MAX_M || N <= 0 || K <= 0 || N > (1 << 24) || K > (1 << 24)) return AMS_ERR_SHAPE;
  if (FMT == FMT_FP16 && (K % 8) != 0) return AMS_ERR_SHAPE;
  if (!aligned16(W) || !aligned16(X) || !aligned16(Y) || (scales && !aligned16(scales))) return AMS_ERR_ALIGN;
  DeviceState* dev = nullptr;
  if (const int rc = device_state(&dev); rc != AMS_OK) return rc;
  const bool static_ws = workspace == kStaticScratch;
  if (static_ws) {  // the library's own scratch, this device's copy
    workspace = dev->scratch;
    ws_bytes = kStaticScratchBytes;
  }
  constexpr int REC_K = Fmt<FMT>::REC_K;
  const int64_t n_strips = (N + 15) / 16;
  const int n_rec = (int)((K + REC_K - 1) / REC_K);
  LinearArgs a;
  a.W = (const uint8_t*)W;
  a.scales = scales;
  a.X = X;
  a.Y = Y;
  a.M = M;
  a.N = (int)N;
  a.K = (int)K;
  a.n_rec = n_rec;
  a.n_strips = (int)n_strips;
  hipStream_t st = (hipStream_t)stream;
  a.n_sg = 0;
  a.sg_shift = 0;
  if (scale_group != 0) {  // one scale per run of scale_group = REC_K * 2^shift input channels
    int shift = -1;
    for (int j = 0; j < 20; j++)
      if (scale_group == (int64_t)REC_K << j) shift = j;
    if (shift < 0 || FMT == FMT_FP16) return AMS_ERR_SHAPE;
    a.sg_shift = shift;
    a.n_sg = (int)((K + scale_group - 1) / scale_group);
  }
  a.gn = 1;
  a.gk = 1;
  a.row_tiles = 1;
  a.tile_rows = M;
  a.wps = 1;
  a.wpa = 1;
  a.ws_tiles = nullptr;
  a.ws_count = nullptr;
  a.red_slots = 0;
  a.piece_q = a.piece_r = 0;
  constexpr int REC_BYTES = FMT == FMT_FP16 ? 4096 : Fmt<FMT>::REC_BYTES;
  Split split = {1, false, {}};
  if (workspace && scale_group == 0) {
    if (!aligned16(workspace)) return AMS_ERR_ALIGN;
    split = choose_split(FMT, M, n_strips, n_rec, REC_K, REC_BYTES, K);
    if (split_workspace_bytes(M, n_strips, split.gk) > ws_bytes) {
      if (static_ws) return AMS_ERR_SCRATCH;  // beyond the static array: refused, never silently another plan
      split = {1, false, {}};                 // a caller's workspace that is too small: no split
    }
  }
  const int gk = split.gk;
  auto use_split = [&](int plan_gk) {
    if (plan_gk > 1) {
      a.ws_count = (unsigned*)workspace;
      a.ws_tiles = (f4*)((uint8_t*)workspace + kSplitCounterBytes);
    }
  };
  if constexpr (FMT != FMT_FP16) {
    // Non-temporal loads for everything but tiny matrices.  Measured with every call reading weights that are not
    // in any cache (a model's layers in turn): equal or up to 5 % faster than ordinary loads at every size; ordinary
    // loads only win when the same few megabytes are read again call after call.
    const bool nt = n_strips * n_rec * (int64_t)REC_BYTES >= (2ll << 20);
    const ColumnPlan cp = split.planned && nt ? split.plan : make_plan(FMT, M, n_strips, n_rec, REC_K, gk, K % 8 == 0, scale_group == 0, nt);
    a.gn = cp.gn;
    a.gk = cp.gk;
    a.row_tiles = cp.row_tiles;
    a.tile_rows = (M + cp.row_tiles - 1) / cp.row_tiles;
    a.wps = cp.wps;
    a.wpa = cp.wpa;
    use_split(cp.gk);
    a.x_stride = cp.x_stride;
    a.x_region = cp.x_region;
    a.x_shift = cp.x_shift;
    a.spw = cp.spw;
    a.rc = cp.rc;
    if (cp.slice) return launch_slice<FMT>(a, cp.variant, cp.rows, cp.spw, cp.grid, st);
    if (cp.ns > 1) return launch_multi<FMT>(a, cp.grid, cp.S, cp.lds, st);
    return M <= 16 ? launch_column<FMT, 1>(nt, scale_group != 0, cp.qd, cp.lr, a, cp.grid, cp.S, cp.lds, st)
                   : launch_column<FMT, 2>(nt, scale_group != 0, cp.qd, cp.lr, a, cp.grid, cp.S, cp.lds, st);
  } else {
    if (const GemvPlan gp = make_gemv_plan(M, K, gk); gp.ok) {
      a.x_stride = gp.kpad;
      const bool nt = N * K * 2 >= (2ll << 20);
      return launch_gemv(M, nt, a, kNumCU, gp.lds, st);
    }
    const SweepPlan wp = make_sweep_plan(FMT, M, n_strips, n_rec, REC_K, false, gk);
    if (wp.ok) {
      a.gn = wp.gn;
      a.gk = wp.gk;
      a.wps = wp.wps;
      use_split(wp.gk);
      a.x_stride = wp.x_stride;
      a.x_region = wp.x_region;
      a.x_shift = wp.x_shift;
      a.spw = wp.spw;
      a.rc = wp.rc;
      return M <= 16 ? launch_fp16<1>(kSweep, wp.lr, a, wp.grid, wp.S, wp.lds, st) : launch_fp16<2>(kSweep, wp.lr, a, wp.grid, wp.S, wp.lds, st);
    }
    const StreamPlan sp = make_stream_plan(FMT, M, n_strips, n_rec, REC_K);
    if (sp.ok) {
      a.x_stride = sp.x_stride;
      a.x_region = sp.x_region;
      a.x_shift = sp.x_shift;
      a.spw = sp.spw;
      a.red_slots = sp.red_slots;
      a.piece_q = (int)(((int64_t)sp.spw * sp.rc) / sp.S);
      a.piece_r = (int)(((int64_t)sp.spw * sp.rc) % sp.S);
      a.rc = sp.rc;
      return M <= 16 ? launch_fp16<1>(kStream, sp.lr, a, sp.grid, sp.S, sp.lds, st) : launch_fp16<2>(kStream, sp.lr, a, sp.grid, sp.S, sp.lds, st);
    }
    return AMS_ERR_SHAPE;  // not reached: the contiguous-piece plan accepts every shape the checks above let through
  }
}

// Raise the LDS limit of every Linear kernel of one weight format on the current device.
template <int FMT>
int prepare_format() {
  LinearArgs a = {};
  bool ok = true;
  if constexpr (FMT != FMT_FP16) {
    for (int r = 4; r <= 32; r *= 2)
      for (int strips = 1; strips <= kSliceMaxStrips; strips++)
        for (int variant = 0; variant < kSliceVariants; variant++)
          if (variant >= kSliceDeep ? slice_has_deep(FMT, variant, r, strips) : variant != kSliceRagged || (r <= kSliceRaggedMaxRows && strips <= kSliceRaggedMaxStrips)) ok &= launch_slice<FMT>(a, variant, r, strips, 0, nullptr) == AMS_OK;
    for (a.K = 8; a.K < 10; a.K++) {  // aligned and ragged rows of X
      for (int nt = 0; nt < 2; nt++)
        for (int gs = 0; gs < 2; gs++)
          for (int qd = 0; qd < 2; qd++) {
            if (gs && (!nt || qd)) continue;
            ok &= launch_column<FMT, 1>(nt, gs, qd, 2, a, 0, 16, 0, nullptr) == AMS_OK;
            ok &= launch_column<FMT, 2>(nt, gs, qd, 2, a, 0, 16, 0, nullptr) == AMS_OK;
          }
      if constexpr (Fmt<FMT>::SG == 1) {
        ok &= launch_multi<FMT>(a, 0, 8, 0, nullptr) == AMS_OK;
        ok &= launch_column<FMT, 1>(true, false, false, 3, a, 0, 8, 0, nullptr) == AMS_OK;
      }
    }
    a.K = 9;
    if constexpr (FMT == FMT_FP425) ok &= launch_column<FMT, 1>(true, false, true, 3, a, 0, 8, 0, nullptr) == AMS_OK;
  } else {
    for (int m = 1; m <= 4; m++)
      for (int nt = 0; nt < 2; nt++) ok &= launch_gemv(m, nt != 0, a, 0, 0, nullptr) == AMS_OK;
    for (int groups = 0; groups < 2; groups++) {
      a.wps = groups ? 8 : 16;
      ok &= launch_fp16<1>(kSweep, 1, a, 0, 16, 0, nullptr) == AMS_OK;
      ok &= launch_fp16<2>(kSweep, 1, a, 0, 16, 0, nullptr) == AMS_OK;
    }
    a.wps = 16;
    ok &= launch_fp16<1>(kSweep, 2, a, 0, 16, 0, nullptr) == AMS_OK;
    ok &= launch_fp16<2>(kSweep, 2, a, 0, 16, 0, nullptr) == AMS_OK;
    for (int lr : {2, 4}) {
      ok &= launch_fp16<1>(kStream, lr, a, 0, 16, 0, nullptr) == AMS_OK;
      ok &= launch_fp16<2>(kStream, lr, a, 0, 16, 0, nullptr) == AMS_OK;
    }
  }
  (void)hipGetLastError();
  return ok ? AMS_OK : AMS_ERR_LAUNCH;
}

}  // namespace

extern "C" {

int ams_init(void) {
  if (const int rc = device_state(); rc != AMS_OK) return rc;
  int rc = prepare_format<FMT_FP533>();
  if (rc == AMS_OK) rc = prepare_format<FMT_FP425>();
  if (rc == AMS_OK) rc = prepare_format<FMT_FP45>();
  if (rc == AMS_OK) rc = prepare_format<FMT_FP433>();
  if (rc == AMS_OK) rc = prepare_format<FMT_FP6>();
  if (rc == AMS_OK) rc = prepare_format<FMT_FP5>();
  if (rc == AMS_OK) rc = prepare_format<FMT_FP4>();
  if (rc == AMS_OK) rc = prepare_format<FMT_FP16>();
  return rc;
}

int ams_linear_static_ws(const void* W_packed, const uint16_t* scales, const uint16_t* X, uint16_t* Y, int M, int64_t N,
                         int64_t K, int fmt, void* stream) {
  switch (fmt) {
    case FMT_FP533: return run_linear<FMT_FP533>(W_packed, scales, X, Y, M, N, K, stream, 0, kStaticScratch, 0);
    case FMT_FP425: return run_linear<FMT_FP425>(W_packed, scales, X, Y, M, N, K, stream, 0, kStaticScratch, 0);
    case FMT_FP45: return run_linear<FMT_FP45>(W_packed, scales, X, Y, M, N, K, stream, 0, kStaticScratch, 0);
    case FMT_FP433: return run_linear<FMT_FP433>(W_packed, scales, X, Y, M, N, K, stream, 0, kStaticScratch, 0);
    case FMT_FP6: return run_linear<FMT_FP6>(W_packed, scales, X, Y, M, N, K, stream, 0, kStaticScratch, 0);
    case FMT_FP5: return run_linear<FMT_FP5>(W_packed, scales, X, Y, M, N, K, stream, 0, kStaticScratch, 0);
    case FMT_FP4: return run_linear<FMT_FP4>(W_packed, scales, X, Y, M, N, K, stream, 0, kStaticScratch, 0);
  }
  return AMS_ERR_FORMAT;
}

int ams_dequant(int fmt, const void* W_packed, const uint16_t* scales, uint16_t* W_out, int64_t N, int64_t K, int scaled,
                void* stream) {
  return ams_dequant_grouped(fmt, W_packed, scales, 0, W_out, N, K, scaled, stream);
}

int ams_dequant_grouped(int fmt, const void* W_packed, const uint16_t* scales, int64_t scale_group, uint16_t* W_out,
                        int64_t N, int64_t K, int scaled, void* stream) {
  const ams::FormatInfo* fi = ams::format_info(fmt);
  if (!fi) return AMS_ERR_FORMAT;
  if (!W_packed || !W_out || (scaled && !scales)) return AMS_ERR_NULL;
  if (N <= 0 || K <= 0 || N > (1 << 24) || K > (1 << 24)) return AMS_ERR_SHAPE;
  if (!aligned16(W_packed)) return AMS_ERR_ALIGN;
  if (const int rc = device_state(); rc != AMS_OK) return rc;
  int sg_shift = -1, n_sg = 0;  // per-row scales
  if (scale_group != 0) {
    for (int j = 0; j < 20; j++)
      if (scale_group == (int64_t)fi->rec_k << j) sg_shift = j;
    if (sg_shift < 0) return AMS_ERR_SHAPE;
    n_sg = (int)((K + scale_group - 1) / scale_group);
  }
  const int n_rec = (int)((K + fi->rec_k - 1) / fi->rec_k);
  const int64_t total = ((N + 15) / 16) * n_rec;
  const unsigned grid = (unsigned)((total + kDequantWaves - 1) / kDequantWaves);
  hipStream_t st = (hipStream_t)stream;
  auto go = [&](auto kern) {
    hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * kDequantWaves), 0, st, (const uint8_t*)W_packed, scales, W_out, (int)N, (int)K, n_rec, total, scaled, n_sg,
                       sg_shift);
  };
  switch (fmt) {
    case FMT_FP533: go(dequant_kernel<FMT_FP533>); break;
    case FMT_FP425: go(dequant_kernel<FMT_FP425>); break;
    case FMT_FP45: go(dequant_kernel<FMT_FP45>); break;
    case FMT_FP433: go(dequant_kernel<FMT_FP433>); break;
    case FMT_FP6: go(dequant_kernel<FMT_FP6>); break;
    case FMT_FP5: go(dequant_kernel<FMT_FP5>); break;
    default: go(dequant_kernel<FMT_FP4>); break;
  }
  return hipGetLastError() == hipSuccess ? AMS_OK : AMS_ERR_LAUNCH;
}

int ams_linear(const void* W_packed, const uint16_t* scales, const uint16_t* X, uint16_t* Y, int M, int64_t N, int64_t K,
               int fmt, void* stream) {
  switch (fmt) {
    case FMT_FP533: return run_linear<FMT_FP533>(W_packed, scales, X, Y, M, N, K, stream);
    case FMT_FP425: return run_linear<FMT_FP425>(W_packed, scales, X, Y, M, N, K, stream);
    case FMT_FP45: return run_linear<FMT_FP45>(W_packed, scales, X, Y, M, N, K, stream);
    case FMT_FP433: return run_linear<FMT_FP433>(W_packed, scales, X, Y, M, N, K, stream);
    case FMT_FP6: return run_linear<FMT_FP6>(W_packed, scales, X, Y, M, N, K, stream);
    case FMT_FP5: return run_linear<FMT_FP5>(W_packed, scales, X, Y, M, N, K, stream);
    case FMT_FP4: return run_linear<FMT_FP4>(W_packed, scales, X, Y, M, N, K, stream);
  }
  return AMS_ERR_FORMAT;
}

int ams_linear_grouped(const void* W_packed, const uint16_t* scales, int64_t scale_group, const uint16_t* X, uint16_t* Y,
                       int M, int64_t N, int64_t K, int fmt, void* stream) {
  if (scale_group <= 0) return AMS_ERR_SHAPE;
  switch (fmt) {
    case FMT_FP533: return run_linear<FMT_FP533>(W_packed, scales, X, Y, M, N, K, stream, scale_group);
    case FMT_FP425: return run_linear<FMT_FP425>(W_packed, scales, X, Y, M, N, K, stream, scale_group);
    case FMT_FP45: return run_linear<FMT_FP45>(W_packed, scales, X, Y, M, N, K, stream, scale_group);
    case FMT_FP433: return run_linear<FMT_FP433>(W_packed, scales, X, Y, M, N, K, stream, scale_group);
    case FMT_FP6: return run_linear<FMT_FP6>(W_packed, scales, X, Y, M, N, K, stream, scale_group);
    case FMT_FP5: return run_linear<FMT_FP5>(W_packed, scales, X, Y, M, N, K, stream, scale_group);
    case FMT_FP4: return run_linear<FMT_FP4>(W_packed, scales, X, Y, M, N, K, stream, scale_group);
  }
  return AMS_ERR_FORMAT;
}

int ams_linear_workspace_bytes(int fmt, int M, int64_t N, int64_t K, size_t* bytes) {
  if (!bytes) return AMS_ERR_NULL;
  if (M < 1 || M > AMS_MAX_M || N <= 0 || K <= 0 || N > (1 << 24) || K > (1 << 24)) return AMS_ERR_SHAPE;
  int rec_k = 128, rec_bytes = 4096, f = FMT_FP16;  // fmt < 0: the fp16 baseline
  if (fmt >= 0) {
    const ams::FormatInfo* fi = ams::format_info(fmt);
    if (!fi) return AMS_ERR_FORMAT;
    rec_k = fi->rec_k, rec_bytes = fi->rec_bytes, f = fmt;
  }
  const int64_t n_strips = (N + 15) / 16;
  const int n_rec = (int)((K + rec_k - 1) / rec_k);
  *bytes = split_workspace_bytes(M, n_strips, choose_split(f, M, n_strips, n_rec, rec_k, rec_bytes, K).gk);
  return AMS_OK;
}

int ams_linear_plan(int fmt, int M, int64_t N, int64_t K, int with_workspace, char* text, size_t text_len) {
  if (!text || text_len == 0) return AMS_ERR_NULL;
  if (M < 1 || M > AMS_MAX_M || N <= 0 || K <= 0 || N > (1 << 24) || K > (1 << 24)) return AMS_ERR_SHAPE;
  int rec_k = 128, rec_bytes = 4096, f = FMT_FP16;
  if (fmt >= 0) {
    const ams::FormatInfo* fi = ams::format_info(fmt);
    if (!fi) return AMS_ERR_FORMAT;
    rec_k = fi->rec_k, rec_bytes = fi->rec_bytes, f = fmt;
  }
  const int64_t n_strips = (N + 15) / 16;
  const int n_rec = (int)((K + rec_k - 1) / rec_k);
  const bool grouped = with_workspace == 2;  // ams_linear_grouped
  const int gk = with_workspace && !grouped ? choose_split(f, M, n_strips, n_rec, rec_k, rec_bytes, K).gk : 1;
  if (f != FMT_FP16) {
    const bool nt = n_strips * n_rec * (int64_t)rec_bytes >= (2ll << 20);  // as run_linear decides it
    const ColumnPlan cp = make_plan(f, M, n_strips, n_rec, rec_k, gk, K % 8 == 0, !grouped, nt);
    if (cp.slice) {
      const int rows = (M + cp.row_tiles - 1) / cp.row_tiles;
      const SliceAsk ask = slice_ask(f, cp.rows, cp.spw, cp.variant);
      size_t len = 0;
      const auto say = [&](const char* format, auto... v) {
        const int n = len < text_len ? snprintf(text + len, text_len - len, format, v...) : 0;
        len += n > 0 ? n : 0;
      };
      say("slice grid=%d strips_per_wg=%d k_slices=%d waves=%d lds=%zu ahead=%d", cp.grid, cp.spw, cp.gk, ask.waves, cp.lds, ask.weights);
      if (ask.streams < ask.waves) say(" streams=%d", ask.streams);
      if (ask.acts > 1) say(" x_ahead=%d", ask.acts);
      if (cp.variant == kSliceRagged)
        say(" streamed_rows=%d row_tiles=%d", rows, cp.row_tiles);
      else if (cp.row_tiles > 1)
        say(" row_tiles=%d rows_per_tile=%d", cp.row_tiles, rows);
    } else {
      snprintf(text, text_len, "column grid=%d strips_per_wg=%d k_slices=%d waves=%d waves_per_strip=%d phases=%d lds=%zu side_groups=%d active_per_strip=%d ahead=%d strips_per_wave=%d", cp.grid,
               cp.spw, cp.gk, cp.S, cp.wps, cp.n_phase, cp.lds, cp.qd ? 1 : 0, cp.ns > 1 ? 1 : cp.wpa, cp.lr, cp.ns);
    }
    return AMS_OK;
  }
  if (const GemvPlan gp = make_gemv_plan(M, K, gk); gp.ok) {
    snprintf(text, text_len, "gemv grid=%d rows_per_wave=%d k_slices=1 waves=16 phases=1 lds=%zu", kNumCU,
             (int)((N + kNumCU * 16 - 1) / (kNumCU * 16)), gp.lds);
    return AMS_OK;
  }
  const SweepPlan wp = make_sweep_plan(f, M, n_strips, n_rec, rec_k, false, gk);
  if (wp.ok) {
    const int slice = (n_rec + gk - 1) / gk;
    snprintf(text, text_len, "sweep grid=%d strips_per_wg=%d k_slices=%d waves=%d waves_per_strip=%d phases=%d lds=%zu", wp.grid, wp.spw,
             wp.gk, wp.S, wp.wps, (slice + wp.rc - 1) / wp.rc, wp.lds);
    return AMS_OK;
  }
  const StreamPlan sp = make_stream_plan(f, M, n_strips, n_rec, rec_k);
  snprintf(text, text_len, "stream grid=%d strips_per_wg=%d k_slices=1 waves=%d phases=%d lds=%zu", sp.grid, sp.spw, sp.S,
           (n_rec + sp.rc - 1) / sp.rc, sp.lds);
  return AMS_OK;
}

int ams_linear_ws(const void* W_packed, const uint16_t* scales, const uint16_t* X, uint16_t* Y, int M, int64_t N, int64_t K,
                  int fmt, void* workspace, size_t workspace_bytes, void* stream) {
  switch (fmt) {
    case FMT_FP533: return run_linear<FMT_FP533>(W_packed, scales, X, Y, M, N, K, stream, 0, workspace, workspace_bytes);
    case FMT_FP425: return run_linear<FMT_FP425>(W_packed, scales, X, Y, M, N, K, stream, 0, workspace, workspace_bytes);
    case FMT_FP45: return run_linear<FMT_FP45>(W_packed, scales, X, Y, M, N, K, stream, 0, workspace, workspace_bytes);
    case FMT_FP433: return run_linear<FMT_FP433>(W_packed, scales, X, Y, M, N, K, stream, 0, workspace, workspace_bytes);
    case FMT_FP6: return run_linear<FMT_FP6>(W_packed, scales, X, Y, M, N, K, stream, 0, workspace, workspace_bytes);
    case FMT_FP5: return run_linear<FMT_FP5>(W_packed, scales, X, Y, M, N, K, stream, 0, workspace, workspace_bytes);
    case FMT_FP4: return run_linear<FMT_FP4>(W_packed, scales, X, Y, M, N, K, stream, 0, workspace, workspace_bytes);
  }
  return AMS_ERR_FORMAT;
}

int ams_fp16_linear_ws(const uint16_t* W, const uint16_t* X, uint16_t* Y, int M, int64_t N, int64_t K, void* workspace,
                       size_t workspace_bytes, void* stream) {
  return run_linear<FMT_FP16>(W, nullptr, X, Y, M, N, K, stream, 0, workspace, workspace_bytes);
}

int ams_fp16_linear(const uint16_t* W, const uint16_t* X, uint16_t* Y, int M, int64_t N, int64_t K, void* stream) {
  return run_linear<FMT_FP16>(W, nullptr, X, Y, M, N, K, stream);
}

int ams_read_probe(const void* buf, size_t bytes, uint32_t* sink, void* stream) {
  if (!buf) return AMS_ERR_NULL;
  if (!aligned16(buf)) return AMS_ERR_ALIGN;
  if (const int rc = device_state(); rc != AMS_OK) return rc;
  const int64_t n_rec = (int64_t)(bytes / 1024);
  // with nothing to read this is an empty launch of the same shape (the launch floor)
  const unsigned grid = n_rec == 0 ? 1u : (unsigned)std::min<int64_t>(kNumCU, (n_rec + 15) / 16);
  if (n_rec == 0)
    hipLaunchKernelGGL(read_probe_kernel, dim3(kNumCU), dim3(1024), 0, (hipStream_t)stream, (const u4*)buf, (int64_t)0, sink);
  else
    hipLaunchKernelGGL(read_probe_kernel, dim3(grid), dim3(1024), 0, (hipStream_t)stream, (const u4*)buf, n_rec, sink);
  return hipGetLastError() == hipSuccess ? AMS_OK : AMS_ERR_LAUNCH;
}

}  // extern "C"
