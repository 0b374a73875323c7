// slice_kernel: the Linear with the activations streamed beside the weights (Sec. 3.3, Sec. 4.2), for
// workgroups of up to eight strips of 16 output channels.  One format per translation unit
// and variant (AMS_SLICE_FMT, AMS_SLICE_RUN_SCALES), so that they compile in parallel.
//
// A workgroup owns NS neighbouring strips and its wavefronts share K: wavefront w takes records w, w + S, ... of all NS
// strips.  The activations of a record are then needed by one wavefront only, so nothing is staged for the
// workgroup and there is no barrier before the sums at the end: a wavefront copies the M x REC_K activations of its
// next record straight into LDS of its own (16 bytes per lane and load, no registers) in the same in-order stream of
// requests as the weights, and one s_waitcnt that counts the younger requests lets a record start as soon as its own
// loads are there (how far ahead it asks: slice_ask).  They arrive in input-channel order; the operand registers are permuted once per record and serve
// all NS strips.  What it replaces staged the activations of all of K (or of a phase of it) for the workgroup, through
// registers, between barriers, and sat in front of the weight stream.
//
// Bound: at M <= 8 by the weight stream and the restoration's VALU work; at larger batches by the one in-order path through
// which a compute unit draws weights (from memory) and activations (from L2), 32 KiB of both in flight: without the activations 4096 x
// 14336 FP4.25 at M = 32 took 9.7 us of 20.2, without weights from memory 14.9, without either 9.0, without the restoration
// 20.1.  So the rows are dealt to several workgroups there (20.3 -> 16.4), and a wavefront asks for one record of activations
// ahead, not two (-> 14.5; the same requests without any work between them take 13.7).
//
// Measured against what it replaced, and with two records of activations ahead / now (us, M = 1 / 4 / 16 / 32): 4096 x 4096 FP4.25
// 5.2 -> 4.3 / 4.1, 6.0 -> 4.5 / 4.2, 7.6 -> 5.8 / 5.3, 13.4 -> 6.8 / 6.1; 4096 x 14336 8.7 -> 8.2 / 7.7, 10.3 -> 8.9 / 8.0, 18.3 -> 12.9 /
// 11.7, 30.9 -> 15.8 / 14.6; 8192 x 8192 FP5.33 10.5 -> 9.8 / 9.6, 11.2 -> 10.0 / 9.8, 15.6 -> 12.9 / 12.0, 25.4 -> 15.5 / 15.1; 28672 x 4096
// FP4.25 12.8 -> 11.7 / 11.5, 13.8 -> 11.9 / 11.8, 15.3 -> 13.6 / 12.8, 21.7 -> 17.0 / 15.5; 256 x 768 4.1 -> 2.4 / 2.3 up to M = 4, 2.8 / 2.4 at 16.
//
// The counted waits need every step to make the same requests in the same order: requests past a wavefront's last record
// are made too, out of the buffers' range (they read no memory), the scheduler may not move requests across the
// barriers below, and every slot of the ring counts as used at the end so that no request is left out as dead.
#include "ams_device.h"

#include <type_traits>

#ifndef AMS_SLICE_FMT
#define AMS_SLICE_FMT 0
#endif
#ifndef AMS_SLICE_RUN_SCALES
#define AMS_SLICE_RUN_SCALES 0
#endif

namespace {
using namespace ams_dev;

__device__ __forceinline__ const void* pointer_of(uint32_t low, uint32_t high) { return (const void*)((uint64_t)high << 32 | low); }

// CHUNK bytes per lane through a buffer descriptor; NT = 2: non-temporal.
template <int CHUNK, int NT = 2>
__device__ __forceinline__ void buffer_load_chunk(uint32_t* w, __amdgpu_buffer_rsrc_t rsrc, int voffset, int soffset) {
  if constexpr (CHUNK == 16) {
    const u4 v = __builtin_amdgcn_raw_buffer_load_b128(rsrc, voffset, soffset, NT);
    w[0] = v[0], w[1] = v[1], w[2] = v[2], w[3] = v[3];
  } else if constexpr (CHUNK == 12) {
    const u3 v = __builtin_amdgcn_raw_buffer_load_b96(rsrc, voffset, soffset, NT);
    w[0] = v[0], w[1] = v[1], w[2] = v[2];
  } else if constexpr (CHUNK == 8) {
    const u2 v = __builtin_amdgcn_raw_buffer_load_b64(rsrc, voffset, soffset, NT);
    w[0] = v[0], w[1] = v[1];
  } else {
    w[0] = __builtin_amdgcn_raw_buffer_load_b32(rsrc, voffset, soffset, NT);
  }
}

// Shape of the kernel for R staged activation rows (4, 8, 16 or 32) and NS strips per workgroup.
template <int FMT, int R, int NS, int VAR>
struct Slice {
  static constexpr bool GS = VAR == kSliceRunScales || VAR == kSliceDeepRuns, RAGGED = VAR == kSliceRagged;
  static constexpr int MT = R > 16 ? 2 : 1;
  static constexpr int RB = R > 16 ? 16 : R;                    // rows of one MFMA tile that are staged
  static constexpr int NI = slice_x_loads(FMT, R), NI1 = NI / MT;  // 1 KiB loads of a record's activations, of one tile's
  static constexpr int BYTES = NI * 1024;
  static constexpr int WL = (Fmt<FMT>::SIDE ? 2 : 1) + GS;      // load instructions of one weight record (and its scales)
  static constexpr SliceAsk ASK = slice_ask(FMT, R, NS, VAR);
  static constexpr int S = ASK.streams, THREADS = 64 * ASK.waves;
  static constexpr bool IDLE = S < ASK.waves;  // some wavefronts only help with the sum at the end
  static constexpr int LX = ASK.acts, LW = ASK.weights, BEHIND = ASK.behind;
  static constexpr int U = NS > LW && !RAGGED ? 1 : NS == 1 ? (LW == 1 ? 2 : 4) : 2;  // records per unrolled round
  // Side dwords that several records share are read by as many wavefronts and stay in the caches (FP4.25, four readers: 4096 x
  // 14336 M = 16 12.7 -> 12.3 us), but for M <= 4 on three strips and more, where they take the weights' place (28672 x 4096 M = 1 11.7, cached 11.9).
  static constexpr int SIDE_NT = Fmt<FMT>::SG == 1 || (R == 4 && NS >= 3) ? 2 : 0;
  static constexpr int RS = U * NS;                             // slots of the weight ring
  static constexpr int ROW = slice_tile_row(S, R, NS), STRIP = slice_tile_strip(S, R, NS);  // floats
  static constexpr int WAVE = slice_wave_lds(FMT, R, NS, VAR);                             // bytes
};

// GS: one scale per run of 2^a.sg_shift records.  A record goes through a fresh tile, times its run's scales, into the
// sum; the four scales of a lane's output channels are one 8-byte load that travels with the record.  28672 x 4096
// FP4.25, a scale per 128: M = 1 15.7 -> 12.8 us, M = 4 15.9 -> 13.5, M = 32 23.5 -> 20.2 (column_kernel before).
//
// RAGGED: rows of X that are not 16-byte aligned (K no multiple of 8) cannot be copied straight into LDS: they are loaded
// one record ahead into registers, 16 unaligned bytes per lane, and written to the wave's own LDS when their record
// begins.  Tiles of up to eight rows and up to four strips, sixteen wavefronts.  us, column_kernel (staged by the workgroup) / here:
// 11003 x 4099 FP5.33 M = 5 10.6 / 8.1, 8192 x 8193 FP4.25 M = 4 12.6 / 9.3, 4096 x 14337 M = 32 47.7 / 22.5.
template <int FMT, int R, int NS, int VAR>
__global__ void __launch_bounds__((Slice<FMT, R, NS, VAR>::THREADS)) slice_kernel(u4 head0, u4 head1, u4 head2, u2 head3, SliceArgs a) {
  const uint8_t* const W = (const uint8_t*)pointer_of(head0[0], head0[1]);
  const uint16_t* const X = (const uint16_t*)pointer_of(head0[2], head0[3]);
  const uint16_t* const scales = (const uint16_t*)pointer_of(head1[0], head1[1]);
  const int M = head1[2], N = head1[3], K = head2[0], n_rec = head2[1], n_strips = head2[2], gn = head2[3], gk_slices = head3[0], tile_rows = head3[1];
  using P = Slice<FMT, R, NS, VAR>;
  constexpr bool GS = P::GS, RAGGED = P::RAGGED;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  constexpr int FAR = kOutOfRange;
  constexpr int REC_K = Fmt<FMT>::REC_K, SG = Fmt<FMT>::SG, NF = Fmt<FMT>::N_MFMA, PB = Fmt<FMT>::PB, UNIT = Fmt<FMT>::UNIT;
  constexpr int MT = P::MT, RB = P::RB, LX = P::LX, LW = P::LW, RS = P::RS, U = P::U, S = P::S;
  static_assert(LW < RS, "weight ring");
  asm volatile("" ::"s"(W), "s"(X), "s"(scales), "s"(M), "s"(K), "s"(n_rec), "s"(n_strips), "s"(gn), "s"(gk_slices));
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Workgroup = (position wg along N and slice of K, row tile of X).  The row tiles of a position read the same weights at
  // the same time: the grid is then rounded up to whole groups of eight along x, which puts them on one XCD and its L2.
  const int wg = blockIdx.x;
  if (wg >= gn * gk_slices) return;
  const int m_first = (int)blockIdx.y * tile_rows;
  const int rows = min(tile_rows, M - m_first);
  const int gk = gk_slices > 1 ? (int)((unsigned)wg / (unsigned)gn) : 0;
  const int s_first = (wg - gk * gn) * NS;
  const int ns = min(NS, n_strips - s_first);
  const int rec_lo = gk_slices > 1 ? (int)((unsigned)(gk * n_rec) / (unsigned)gk_slices) : 0;
  const int rec_hi = gk_slices > 1 ? (int)((unsigned)((gk + 1) * n_rec) / (unsigned)gk_slices) : n_rec;
  const int first = rec_lo + wave;  // this wave's records: first, first + S, ...
  const int cnt = (!P::IDLE || wave < S) && first < rec_hi ? (rec_hi - first + S - 1) / S : 0;
  // The scales of the workgroup's channels are asked for ahead of the stream and not touched before its end.  (Behind a
  // branch, the compiler moved their conversion up to the load: the first wavefront then waited for memory before its
  // first record.)  Threads beyond them, and channels beyond N, ask for nothing and get 0.
  uint32_t scale_bits = 0x3C00;
  if (!GS && wave < (NS * 16 + 63) / 64) {
    const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)scales, 0, N * 2, 0x00020000);
    scale_bits = __builtin_amdgcn_raw_buffer_load_b16(rs, tid < NS * 16 ? (s_first * 16 + tid) * 2 : FAR, 0, 0);
  }
  __builtin_amdgcn_sched_barrier(0);

  f4 acc[NS][MT];
#pragma unroll
  for (int i = 0; i < NS; i++)
#pragma unroll
    for (int t = 0; t < MT; t++) acc[i][t] = f4{0, 0, 0, 0};

  if (cnt > 0) {
    unsigned char* const xbuf = smem + wave * P::WAVE;
    // A load brings 16 (8, 4) rows x 4 (8, 16) pieces of 16 bytes: four neighbouring lanes read 64 neighbouring bytes of a
    // row (with neighbouring lanes in different rows the same bytes take three times as long).  The pieces of four lanes
    // are swapped by a function of the row that makes the reads of an operand, 8 or 16 rows at one piece, free of bank
    // conflicts; LDS takes them in lane order.
    auto swz = [](int m) { return ((m >> 2) & 1) | ((((m >> 1) ^ (m >> 3)) & 1) << 1); };
    // loads: lane -> row, block of four pieces, piece
    constexpr int BLK = 64 / (4 * RB);  // blocks of four pieces per load
    const int ld_m = (lane >> 2) & (RB - 1), ld_b = lane / (4 * RB);
    // Requests past the wave's last record (p >= cnt) get an offset out of the buffer's range: they read no memory but
    // count like the others.  (The scalar offset always stays inside the buffer: only the vector part is out of range.)
    const int row_bytes = K * 2;
    // Lanes whose row does not exist, or whose block lies behind the record, ask for nothing (FAR, below): what they would
    // bring takes cache lines from the weight stream.
    int voff[MT], voff_last[MT];
#pragma unroll
    for (int t = 0; t < MT; t++) {
      const int off = (16 * t + ld_m) * row_bytes + ld_b * 64 + (((lane & 3) ^ swz(ld_m)) * 16);
      voff[t] = 16 * t + ld_m < rows ? off : FAR;
      voff_last[t] = P::NI1 * BLK == REC_K / 32 || ld_b + (P::NI1 - 1) * BLK < REC_K / 32 ? voff[t] : FAR;
    }
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)(X + (size_t)m_first * K), 0, rows * row_bytes, 0x00020000);
    // reads: operand u of this lane's activation row
    const int m_lo = lane & (RB - 1), kq = lane >> 4;
    int roff[NF];
#pragma unroll
    for (int u = 0; u < NF; u++) {
      const int piece = kq * NF + u;
      roff[u] = (piece >> 2) * (RB * 64) + m_lo * 64 + (((piece & 3) ^ swz(m_lo)) * 16);
    }
    // RAGGED: the loads' rows, the channels of their pieces inside a record, and the record under way.  Lanes whose row does
    // not exist ask for nothing on tiles of eight rows, and for row 0 on tiles of four, where the branch costs one and three
    // rows 2-3 %.  (With the last row again for all of them its lines were asked for by lanes in several pairs of rows,
    // which takes longer the more there are: 2544 x 6015 FP4.33, 2 / 6 / 10 rows 6.6 / 8.8 / 10.1 us, now 5.4 / 7.7 / 8.5.)
    int row_at[MT], piece_at[MT];
    u4 ahead[RAGGED ? P::NI : 1] = {};
    if constexpr (RAGGED) {
#pragma unroll
      for (int t = 0; t < MT; t++) {
        row_at[t] = (16 * t + ld_m < rows ? 16 * t + ld_m : 0) * K;
        piece_at[t] = ld_b * 32 + ((lane & 3) ^ swz(ld_m)) * 8;
      }
    }
    const uint16_t* const xrows = X + (size_t)m_first * K;
    auto request_ragged = [&](int p) {
      const int rec = p < cnt ? first + S * p : first;  // behind the last record: any record (the results are not used)
#pragma unroll
      for (int t = 0; t < MT; t++)
#pragma unroll
        for (int i = 0; i < P::NI1; i++)  // a piece that runs past its row's end: the row's last eight channels
          if (RB == 4 || 16 * t + ld_m < rows) __builtin_memcpy(&ahead[t * P::NI1 + i], xrows + row_at[t] + min(rec * REC_K + piece_at[t] + i * (BLK * 32), K - 8), 16);
    };
    auto store_ragged = [&](int p) {
      const int rec = first + S * p;
#pragma unroll
      for (int t = 0; t < MT; t++)
#pragma unroll
        for (int i = 0; i < P::NI1; i++) {
          u4 v = ahead[t * P::NI1 + i];
          if (rec == n_rec - 1) {  // channels beyond K count as zero
            const int beyond = rec * REC_K + piece_at[t] + i * (BLK * 32) + 8 - K;
            uint32_t h[4] = {v[0], v[1], v[2], v[3]};
            shift_tail(h, beyond);
            const uint32_t keep = beyond < 8 ? 0xFFFFFFFFu : 0u;
            v = u4{h[0] & keep, h[1] & keep, h[2] & keep, h[3] & keep};
          }
          *(u4*)(xbuf + (t * P::NI1 + i) * 1024 + lane * 16) = v;
        }
    };
    auto request_x = [&](int p) {  // the wave's p-th record of activations
      const int soff = p < cnt ? (first + S * p) * (REC_K * 2) : 0;
      unsigned char* dst = xbuf + (p & (LX - 1)) * P::BYTES;
#pragma unroll
      for (int t = 0; t < MT; t++)
#pragma unroll
        for (int i = 0; i < P::NI1; i++) {
          const int vo = p < cnt ? (i == P::NI1 - 1 ? voff_last[t] : voff[t]) + i * (BLK * 64) : FAR;
          __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (__attribute__((address_space(3))) void*)(dst + (t * P::NI1 + i) * 1024), 16, vo, soff, 0, 0);
        }
    };
    struct Scales {
      uint32_t h[2];  // four halfs
    };
    LaneRec<FMT> ring[RS];
    Scales ring_sc[GS ? RS : 1];
    auto request_w = [&](int p, int i, LaneRec<FMT>& slot, Scales& sc) {  // the weights of strip i for the wave's p-th record
      const unsigned rec = p < cnt ? (first + S * p) : 0;
      const uint8_t* unit = W + ((size_t)(rec / SG) * (unsigned)n_strips + (unsigned)(s_first + min(i, ns - 1))) * UNIT;
      const __amdgpu_buffer_rsrc_t w = __builtin_amdgcn_make_buffer_rsrc((void*)unit, 0, UNIT, 0x00020000);
      const int vo = p < cnt ? lane * Fmt<FMT>::CHUNK : FAR;
      buffer_load_chunk<Fmt<FMT>::CHUNK>(slot.w, w, vo, (int)(rec % SG) * Fmt<FMT>::CB);
      if constexpr (Fmt<FMT>::SIDE != 0) {
        const int vs = p < cnt ? lane * 4 : FAR;
        buffer_load_chunk<4, P::SIDE_NT>(&slot.t, w, vs, SG * Fmt<FMT>::CB);
      }
      if constexpr (GS) {  // cached: a run spans many records and rows of lanes
        const uint16_t* run = scales + ((size_t)(s_first + min(i, ns - 1)) * a.n_sg + (rec >> a.sg_shift)) * 16;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)run, 0, 32, 0x00020000);
        const int vg = p < cnt ? kq * 8 : FAR;
        buffer_load_chunk<8, 0>(sc.h, rs, vg, 0);
      }
    };
    const int tail = n_rec * REC_K - K;  // channels of the last record beyond K

    // One record of all strips.  uc: its place in the unrolled round.  The wait lets through exactly the loads requested
    // after this record's activations: every step makes the same requests, those past the end out of range.
    auto step = [&](int p, auto uc) {
      constexpr int u0 = decltype(uc)::value * NS;  // its first slot of the ring
      // younger than record p's activations when step p begins: the weights requested since, and the records behind it
      constexpr int STEADY = (LX * NS - P::BEHIND) * P::WL + (LX - 1) * P::NI;
      constexpr auto at_start = [](int q) { return (LW + q * NS < LX * NS - P::BEHIND ? LW + q * NS : LX * NS - P::BEHIND) * P::WL + (LX - 1) * P::NI; };
      if constexpr (RAGGED) {
        store_ragged(p);  // the compiler sees the loads and waits for them itself
        request_ragged(p + 1);
        __builtin_amdgcn_sched_barrier(0);
      } else if constexpr (LW >= LX * NS - P::BEHIND) {
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(STEADY) : "memory");
      } else {  // the first steps have fewer weights requested behind their activations
        if (p == 0)
          asm volatile("s_waitcnt vmcnt(%0)" ::"n"(at_start(0)) : "memory");
        else if (LX > 1 && p == 1)
          asm volatile("s_waitcnt vmcnt(%0)" ::"n"(at_start(1)) : "memory");
        else
          asm volatile("s_waitcnt vmcnt(%0)" ::"n"(STEADY) : "memory");
      }
      u4 b[MT][NF];
      const unsigned char* src = RAGGED ? xbuf : xbuf + (p & (LX - 1)) * P::BYTES;
#pragma unroll
      for (int t = 0; t < MT; t++)
#pragma unroll
        for (int u = 0; u < NF; u++) b[t][u] = *(const u4*)(src + t * (P::NI1 * 1024) + roff[u]);
      if constexpr (!RAGGED) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (P::BEHIND == 0) request_x(p + LX);
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
      }
      const int rec = (first + S * p);
      if (!RAGGED && tail != 0 && rec == n_rec - 1) {  // channels beyond K: whatever was read there counts as zero
#pragma unroll
        for (int u = 0; u < NF; u++) {
          const uint32_t keep = rec * REC_K + (kq * NF + u) * 8 < K ? 0xFFFFFFFFu : 0u;
#pragma unroll
          for (int t = 0; t < MT; t++) b[t][u] &= u4{keep, keep, keep, keep};
        }
      }
      // into operand order
#pragma unroll
      for (int t = 0; t < MT; t++)
#pragma unroll
        for (int blk = 0; blk < NF * 8 / PB; blk++) {
          uint32_t in[PB / 2], out[PB / 2];
#pragma unroll
          for (int e = 0; e < PB / 2; e++) in[e] = b[t][blk * (PB / 8) + e / 4][e % 4];
          permute_unit<FMT>(in, out);
#pragma unroll
          for (int e = 0; e < PB / 2; e++) b[t][blk * (PB / 8) + e / 4][e % 4] = out[e];
        }
      const int side_shift = 8 * Fmt<FMT>::SIDE * (rec & (SG - 1));
#pragma unroll
      for (int i = 0; i < NS; i++) {
        request_w(p + (i + LW) / NS, (i + LW) % NS, ring[(u0 + i + LW) % RS], ring_sc[GS ? (u0 + i + LW) % RS : 0]);
        if (!RAGGED && i == P::BEHIND - 1) {
          __builtin_amdgcn_sched_barrier(0);
          asm volatile("" ::: "memory");
          request_x(p + LX);
          asm volatile("" ::: "memory");
        }
        __builtin_amdgcn_sched_barrier(0);
        uint32_t o[4 * NF];
        restore_rec<FMT>(ring[u0 + i], side_shift, o);
        f4 own[MT];  // GS: this record's tile
        if constexpr (GS) {
#pragma unroll
          for (int t = 0; t < MT; t++) own[t] = f4{0, 0, 0, 0};
        }
#pragma unroll
        for (int u = 0; u < NF; u++) {
          const h8 w = __builtin_bit_cast(h8, u4{o[4 * u], o[4 * u + 1], o[4 * u + 2], o[4 * u + 3]});
#pragma unroll
          for (int t = 0; t < MT; t++) {
            f4& c = GS ? own[t] : acc[i][t];
            c = __builtin_amdgcn_mfma_f32_16x16x32_f16(w, __builtin_bit_cast(h8, b[t][u]), c, 0, 0, 0);
          }
        }
        if constexpr (GS) {
          const Scales h = ring_sc[u0 + i];
          f4 sc;
#pragma unroll
          for (int r = 0; r < 4; r++) sc[r] = (float)__builtin_bit_cast(_Float16, (uint16_t)(h.h[r >> 1] >> (16 * (r & 1))));
#pragma unroll
          for (int t = 0; t < MT; t++) acc[i][t] += own[t] * sc;
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    using std::integral_constant;
    if constexpr (RAGGED) {
      static_assert(LX == 1, "one record under way");
      request_ragged(0);
    } else {
#pragma unroll
      for (int q = 0; q < LX; q++) request_x(q);
    }
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < LW; q++) {
      request_w(q / NS, q % NS, ring[q], ring_sc[GS ? q : 0]);
      __builtin_amdgcn_sched_barrier(0);
    }
    int p = 0;
    for (; p + U <= cnt; p += U) {
      step(p, integral_constant<int, 0>{});
      if constexpr (U > 1) step(p + 1, integral_constant<int, 1>{});
      if constexpr (U > 2) step(p + 2, integral_constant<int, 2>{});
      if constexpr (U > 3) step(p + 3, integral_constant<int, 3>{});
    }
    if constexpr (U > 1)
      if (p < cnt) step(p, integral_constant<int, 0>{});
    if constexpr (U > 2)
      if (p + 1 < cnt) step(p + 1, integral_constant<int, 1>{});
    if constexpr (U > 3)
      if (p + 2 < cnt) step(p + 2, integral_constant<int, 2>{});
    // The waits above count on every request: none may be left out as unused.
#pragma unroll
    for (int q = 0; q < RS; q++) {
      asm volatile("" ::"v"(ring[q].w[0]));
      if constexpr (Fmt<FMT>::SIDE != 0) asm volatile("" ::"v"(ring[q].t));
      if constexpr (GS) asm volatile("" ::"v"(ring_sc[q].h[0]));
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the requests past the end are done with LDS
  }
  asm volatile("" : "+v"(scale_bits));
  // Partial tiles [wave][strip][activation row][16 channels, padded], each wavefront's where its own activations were, then
  // the scales, then who was last.
  float* const parts = (float*)smem;
  float* const scale_of = (float*)(smem + S * P::WAVE);
  int* const last = (int*)(scale_of + NS * 16);
  {
    const int m_lo = lane & 15, kq = lane >> 4;
    if (m_lo < RB && (!P::IDLE || wave < S))
#pragma unroll
      for (int i = 0; i < NS; i++)
#pragma unroll
        for (int t = 0; t < MT; t++) *(f4*)(parts + wave * (P::WAVE / 4) + i * P::STRIP + (16 * t + m_lo) * P::ROW + 4 * kq) = acc[i][t];
  }
  if (tid < NS * 16) scale_of[tid] = (float)__builtin_bit_cast(_Float16, (uint16_t)scale_bits) * kTwo14;
  __syncthreads();
  uint16_t* const Y = a.Y + (size_t)m_first * N;
  const int pairs = rows * NS;
  // Four neighbouring channels of an output row: the wavefronts' sums added in wave order; what leaves for Y.
  auto quad_sum = [&](int i, int m, int c) {
    f4 sum = f4{0, 0, 0, 0};
#pragma unroll
    for (int w = 0; w < S; w++) sum += *(const f4*)(parts + w * (P::WAVE / 4) + i * P::STRIP + m * P::ROW + c);
    return sum;
  };
  auto finish_quad = [&](int i, int m, int c, const f4 sum) {
    const int row = (s_first + i) * 16 + c;
    us4 h;
#pragma unroll
    for (int r = 0; r < 4; r++) h[r] = __builtin_bit_cast(uint16_t, (_Float16)(sum[r] * scale_of[i * 16 + c + r]));
    if ((N & 3) == 0) {  // whole quads of channels, eight aligned bytes of Y's row
      if (row < N) *(us4*)(Y + (size_t)m * N + row) = h;
    } else {
#pragma unroll
      for (int r = 0; r < 4; r++)
        if (row + r < N) Y[(size_t)m * N + row + r] = h[r];
    }
  };
  if (gk_slices == 1) {
    // With many outputs a quad per thread: 28672 x 4096 FP5.33 M = 32 20.4 -> 19.9 us, 20000 x 2048 FP4.25 M = 24 9.2 -> 8.9.  With few,
    // more threads share them: 4096 x 4096 M = 9 5.33, as quads 5.51; three strips as quads 1-4 % slower up to 12 rows (10569 x
    // 264 FP5.33 M = 9 3.46 / 3.65), equal at 13.
    constexpr bool QUADS = R >= 16 && NS >= 3;
    if (QUADS && (R > 16 || NS > 3 || pairs >= 40)) {
      for (int u = tid; u < pairs * 4; u += P::THREADS) {
        const int c = 4 * (u & 3), i = (u >> 2) % NS, m = (u >> 2) / NS;
        finish_quad(i, m, c, quad_sum(i, m, c));
      }
    } else {  // one output per thread
      const int n = tid & 15;
      for (int p = tid >> 4; p < pairs; p += P::THREADS / 16) {
        const int i = p % NS, m = p / NS, row = (s_first + i) * 16 + n;
        float sum = 0;
#pragma unroll
        for (int w = 0; w < S; w++) sum += parts[w * (P::WAVE / 4) + i * P::STRIP + m * P::ROW + n];
        if (row < N) Y[(size_t)m * N + row] = __builtin_bit_cast(uint16_t, (_Float16)(sum * scale_of[i * 16 + n]));
      }
    }
    return;
  }
  // K is split over gk workgroups: the same exchange as exchange_tile's, with the workgroup's barriers around the count
  // (every wave's stores are acknowledged before any strip is counted in).  Quads of channels, and the slices' tiles are all
  // asked for before the first is added: one by one they were a trip to memory each (5120 x 25600 FP5.33 M = 16, four slices,
  // 22.9 -> 19.4 us; 4096 x 14336 FP4.25 M = 32 18.0 -> 13.6).
  const int tile = M > 16 ? 512 : 256;  // floats of a strip's tile: the rows of all row tiles
  unsigned* const counts = a.ws_count + s_first * a.row_tiles + blockIdx.y;  // of this row tile: one per strip
  const __amdgpu_buffer_rsrc_t tiles = __builtin_amdgcn_make_buffer_rsrc((void*)a.ws_tiles, 0, gk_slices * n_strips * tile * 4, 0x00020000);
  auto tile_offset = [&](int slice, int i, int m, int c) { return (((slice * n_strips + s_first + i) * tile) + (m_first + m) * 16 + c) * 4; };
  for (int u = tid; u < pairs * 4; u += P::THREADS) {
    const int c = 4 * (u & 3), i = (u >> 2) % NS, m = (u >> 2) / NS;
    const f4 sum = quad_sum(i, m, c);
    if (i < ns) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u4, sum), tiles, tile_offset(gk, i, m, c), 0, kDeviceScope);
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid < ns) {
    const unsigned before = __hip_atomic_fetch_add(counts + tid * a.row_tiles, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const bool is_last = before == (unsigned)gk_slices - 1;
    if (is_last) __hip_atomic_store(counts + tid * a.row_tiles, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    last[tid] = is_last;
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  for (int u = tid; u < pairs * 4; u += P::THREADS) {
    const int c = 4 * (u & 3), i = (u >> 2) % NS, m = (u >> 2) / NS;
    if (i >= ns || !last[i]) continue;
    f4 part[kMaxSlices];
#pragma unroll
    for (int q = 0; q < kMaxSlices; q++) part[q] = f4{0, 0, 0, 0};
    auto request = [&](int q) {  // slices that do not exist read nothing and add 0
      part[q] = __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(tiles, q < gk_slices ? tile_offset(q, i, m, c) : FAR, 0, kDeviceScope));
    };
    request(0), request(1);
    if (gk_slices > 2) request(2), request(3);
    if (gk_slices > 4) request(4), request(5), request(6), request(7);
    f4 sum = f4{0, 0, 0, 0};
#pragma unroll
    for (int q = 0; q < kMaxSlices; q++) sum += part[q];
    finish_quad(i, m, c, sum);
  }
}

template <int V, int R>
const void* by_strips(int strips) {
  constexpr int F = AMS_SLICE_FMT;
  switch (strips) {
    case 1: return (const void*)slice_kernel<F, R, 1, V>;
    case 2: return (const void*)slice_kernel<F, R, 2, V>;
    case 3: return (const void*)slice_kernel<F, R, 3, V>;
    case 4: return (const void*)slice_kernel<F, R, 4, V>;
  }
  if constexpr (V != kSliceRagged) {
    switch (strips) {
      case 5: return (const void*)slice_kernel<F, R, 5, V>;
      case 6: return (const void*)slice_kernel<F, R, 6, V>;
      case 7: return (const void*)slice_kernel<F, R, 7, V>;
      case 8: return (const void*)slice_kernel<F, R, 8, V>;
    }
  }
  return nullptr;
}
template <int V>
const void* by_rows(int rows, int strips) {
  switch (rows) {
    case 4: return by_strips<V, 4>(strips);
    case 8: return by_strips<V, 8>(strips);
  }
  if constexpr (V != kSliceRagged) {
    switch (rows) {
      case 16: return by_strips<V, 16>(strips);
      case 32: return by_strips<V, 32>(strips);
    }
  }
  return nullptr;
}

template <int V>
const void* by_rows_deep(int rows, int strips) {
  constexpr int F = AMS_SLICE_FMT;
  if constexpr (slice_has_deep(F, V, 4, 1))
    if (rows == 4 && strips == 1) return (const void*)slice_kernel<F, 4, 1, V>;
  if constexpr (slice_has_deep(F, V, 16, 1))
    if (rows == 16 && strips == 1) return (const void*)slice_kernel<F, 16, 1, V>;
  return nullptr;
}

}  // namespace

#if AMS_SLICE_RUN_SCALES
template <>
const void* ams_dev::slice_kernel_of<AMS_SLICE_FMT, ams_dev::kSliceRunScales>(int rows, int strips) {
  return by_rows<kSliceRunScales>(rows, strips);
}
template <>
const void* ams_dev::slice_kernel_of<AMS_SLICE_FMT, ams_dev::kSliceDeepRuns>(int rows, int strips) {
  return by_rows_deep<kSliceDeepRuns>(rows, strips);
}
#else
template <>
const void* ams_dev::slice_kernel_of<AMS_SLICE_FMT, ams_dev::kSlicePlain>(int rows, int strips) {
  return by_rows<kSlicePlain>(rows, strips);
}
template <>
const void* ams_dev::slice_kernel_of<AMS_SLICE_FMT, ams_dev::kSliceRagged>(int rows, int strips) {
  return by_rows<kSliceRagged>(rows, strips);
}
template <>
const void* ams_dev::slice_kernel_of<AMS_SLICE_FMT, ams_dev::kSliceDeep>(int rows, int strips) {
  return by_rows_deep<kSliceDeep>(rows, strips);
}
#endif
