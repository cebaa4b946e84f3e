// forward_steps over a buffer of frames as one implicit GEMM over time
// (groups = 1), for the layers of the GEMM families.
//
// A step contracts one frame; a buffer of T frames holds all the taps of most
// of the outputs it completes, so those outputs need no partial sums at all:
// output tau of stream b is the sum over the temporal taps j, the spatial
// taps and the channels of W_j x frame (tau sT + j dT), and every output is
// independent of the others.  The GEMM's rows are the output pixels of one
// stream, all its frames in a row (m = frame * Ho * Wo + pixel, which is the
// order of y), its columns the output channels, its depth K = (temporal tap,
// then the step kernel's own order of spatial taps and channel blocks).
// Outputs whose first frames came before the call start from their partial
// sum in the ring; outputs that the call does not complete end in the ring.
// Each output thus sees the same matrix instructions on the same operands in
// the same order as single steps give it, with its accumulator in registers
// instead of the ring between them, so the results equal stepping bit for bit.
// The weights are read as the step kernels packed them.
//
// Against one persistent workgroup per output tile that walks the frames one
// by one, the time axis gives the chip T times as many tiles, no frame waits
// for the one before it, and a tile's K loop is kT times as long.
//
// Workgroup: M_WG pixels x N_WG channels, wave tiles of 64 pixels x 16 WNF
// channels.  Per k-step (a spatial tap and a block of 32 bf16 or 16 fp32
// channels) the workgroup gathers the pixels' channels, eight (four) of one
// pixel per 16-byte LDS unit, one or two k-steps ahead in registers and double
// buffered in LDS; the weights go from L2 straight to the registers of the
// waves that use them, one k-step ahead.  Units are swizzled by pixel so that
// 8 lanes' operand reads fall into distinct banks.
//
// Up to three workgroups share a CU (two where their registers or the window
// below need it): a workgroup's prologue, barriers and epilogue are long against
// its K loop, and with one resident workgroup of eight waves the same tiles took
// half as long again (192 -> 432 channels, 1x1x1, 7x7, 16 streams, 64 frames: 45
// us against 31 us).  That layer is then bound by the round trips of its
// workgroups, 2000 of six k-steps each: the pixels' gather, a barrier a k-step
// and the epilogue; the weights' way through L1 (4 KB for 16 matrix
// instructions of a 64 x 64 wave tile) is about 4 us of it.  float32 is bound by
// its matrix instructions while the CUs have a workgroup each, and after that by
// the second pass of the workgroups that own ring slots (about 41 of 227 us in
// the layer below, 32 workgroups of 480).
//
// Measured against single steps: the pointwise layer 455 -> 31 us; 128 -> 128,
// (9,1), 25 joints, 16 streams, 150 frames, float32 839 -> 227 us; 64 -> 64 bf16,
// 32 streams, 300 frames 2264 -> 44 us.
//
// The ring.  Output tau's partial sum lives in slot tau mod R, and an output
// that the call leaves unfinished may take the slot of one that it completes.
// The workgroups that own the first R outputs' pixels therefore make a second
// pass: the same pixels of the unfinished outputs of the same slots, after
// their first pass has read them.  A ring element is read and written by one
// lane.
#include <algorithm>
#include <type_traits>

#include "device.hpp"
#include "launch.hpp"

namespace coinf {

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));


// LDS of a window (WINDOW below): two workgroups per CU.
constexpr int kClipWindowBytes = 80 * 1024;

// A call frame that no tap moves into the call.
constexpr int kNoFrame = -(1 << 29);

enum ClipPack : int32_t { kPackReg = 0, kPackGemm = 1, kPackWs = 2 };

struct ClipArgs : FrameSpan {
  int32_t shift;     // pixels by which the tiles begin early (see PAIR)
  int32_t m_pairs, n_tiles;  // (pixel tile, stream) pairs; channel tiles
  int32_t y_bytes, w_bytes, ring_bytes;
  int32_t plane;     // elements between input channels
  int32_t span;      // of them, the call's: T * S
  int32_t y_bc;      // elements between output channels
  int32_t ring_slot;
  int32_t nq, ntaps;  // k-steps per temporal tap; spatial taps
  int32_t tap_outer; // spatial taps outside channel blocks (else inside)
  int32_t pack, wcols, wq;  // weight packing: its column tile, bytes between k-steps
  int32_t wtile;     // bytes between column tiles (or 16-column fragments)
  int32_t tap_cols;  // C_out modulo the column tile
  int32_t tap_bytes;  // (0:) from a tap's last k-step to the next tap's first
  int32_t cgrp;      // channels between lane groups
  uint32_t celt;     // bytes between a 16-byte unit's channels (at most 2^31)
  int32_t act;
  int32_t unpadded;  // one spatial tap, no padding: every pixel's lies in its plane
  int32_t win_rows;  // WINDOW: staged pixels, a multiple of 128
  FastDiv fd_nrb, fd_B, fd_nt, fd_So, fd_Wo, fd_R, fd_q, fd_kW, fd_wcols, fd_dT;
};

template <typename T>
struct ClipFrag;
template <>
struct ClipFrag<bf16_t> {
  using type = v8bf;
};
template <>
struct ClipFrag<float> {
  using type = v4f;
};

__device__ __forceinline__ void clip_mma(v4f& acc, const v8bf& a, const v8bf& b, int) {
  acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, acc, 0, 0, 0);
}
__device__ __forceinline__ void clip_mma(v4f& acc, const v4f& a, const v4f& b, int i) {
  acc = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[i], acc, 0, 0, 0);
}

// Eight channels of a pixel pair (first pixel in the low halves) as the two
// pixels' units.
__device__ __forceinline__ void pair_units(const uint32_t (&r)[8], uint4& u0, uint4& u1) {
  auto lo = [](uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x05040100u); };
  auto hi = [](uint32_t a, uint32_t b) { return __builtin_amdgcn_perm(b, a, 0x07060302u); };
  u0 = make_uint4(lo(r[0], r[1]), lo(r[2], r[3]), lo(r[4], r[5]), lo(r[6], r[7]));
  u1 = make_uint4(hi(r[0], r[1]), hi(r[2], r[3]), hi(r[4], r[5]), hi(r[6], r[7]));
}
__device__ __forceinline__ void pair_units(const uint32_t (&)[4], uint4&, uint4&) {}

// PAIR (bf16, one spatial tap, temporal stride 1): two consecutive pixels are
// consecutive in every input plane, so one 4-byte load (at any 2-byte
// alignment) brings a channel of both.  In the second pass they are, too,
// except where the slots wrap around to the first unfinished output: when that
// is an odd pixel, the tiles begin one pixel early so that no pair spans it.
//
// FAR: a k-step reaches past C_in by up to its width, and with few channels of
// many frames those channels' offsets would pass 2^32 and begin again inside
// the stream, so channel offsets are scalar and stop at the stream's end.  Only
// for the calls that need it: where few workgroups share the chip, adding the
// offsets lane by lane is faster (96 -> 96, 3x3x3, 14x14, bf16, 16 frames: 98
// us against 106; float32 64 -> 64, (9,1), 25 joints: 55.5 against 58).
template <typename T, int WMF, int WNF, int NWM, int NWN, bool PAIR, bool WINDOW, bool FAR>
__global__ __launch_bounds__(64 * NWM * NWN, WMF * WNF > (WINDOW ? 8 : 16) ? 2 : 3) void conv_clip_gemm_kernel(
    ConvGeom g, ClipArgs ca, const T* __restrict__ x, T* __restrict__ y,
    const uint4* __restrict__ wp, const float* __restrict__ bias, float* __restrict__ ring) {
  using Frag = typename ClipFrag<T>::type;
  constexpr int KL = 16 / int(sizeof(T));  // channels per 16-byte unit
  constexpr int CK = 4 * KL;               // channels per k-step
  // stages (k-steps) by which the gathers run ahead
  constexpr int PD = PAIR && WNF < 4 ? 2 : 1;
  constexpr int UN = PD < 2 ? 2 : PD;  // stages per turn of the K loop
  constexpr int NW = NWM * NWN;
  constexpr int M_WG = 16 * WMF * NWM, N_WG = 16 * WNF * NWN;
  constexpr int PXB = PAIR ? 128 : 64;     // pixels of one wave's load
  constexpr int MB = M_WG / PXB;
  constexpr int ITEMS = 4 * MB / NW;       // staging items per wave and stage
  constexpr int NBLK = (4 * MB + NW - 1) / NW;  // pixel blocks a wave stages
  constexpr int esz = int(sizeof(T));
  static_assert(!WINDOW || (PAIR && NW == 4), "window staging");
  static_assert(!(FAR && PAIR), "channel offsets");
  extern __shared__ uint4 clip_lds[];
  uint4(*As)[M_WG * 4] = reinterpret_cast<uint4(*)[M_WG * 4]>(clip_lds);

  const int tid = int(threadIdx.x);
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lrow = lane & 15, lgrp = lane >> 4;
  const int wm = wave / NWN, wn = wave % NWN;

  // Blocks are dealt to the 8 XCDs in turn: the channel tiles of one pixel
  // tile run on one XCD, one after the other, and share its input in L2.
  const int bid = int(blockIdx.x) >> 3;
  const int bp = fdiv(bid, ca.fd_nt);
  const int nt = bid - bp * ca.n_tiles;
  const int pair = bp * 8 + (int(blockIdx.x) & 7);
  if (pair >= ca.m_pairs) return;  // whole workgroups
  const int mt = fdiv(pair, ca.fd_B), b = pair - mt * g.B;
  const int m0 = mt * M_WG - ca.shift;  // (the first tile may begin with one pixel too few)

  // the stream's planes only: channels past C_in read out of range (zero)
  const int x_bytes = ((g.Cin - 1) * ca.plane + ca.span) * esz;
  const __amdgpu_buffer_rsrc_t xr = make_rsrc(x + int64_t(b) * g.Cin * ca.plane, x_bytes);
  const __amdgpu_buffer_rsrc_t yr = make_rsrc(y, ca.y_bytes);
  const __amdgpu_buffer_rsrc_t rr = make_rsrc(ring, ca.ring_bytes);
  const __amdgpu_buffer_rsrc_t br = make_rsrc(bias, g.Cout * 4);

  // this lane's output channel in fragment f
  auto oc = [&](int f) { return nt * N_WG + (wn * WNF + f) * 16 + lrow; };

  // this lane's weight columns n = j C_out + oc at temporal tap j.  Where
  // C_out is whole column tiles, the taps differ by a uniform offset only.
  int woff[WNF];
  auto weight_cols = [&](int j) __attribute__((always_inline)) {
#pragma unroll
    for (int f = 0; f < WNF; ++f) {
      const int n = j * g.Cout + oc(f);
      const int tile = fdiv(n, ca.fd_wcols), nl = n - tile * ca.wcols;
      const int in = ca.pack == kPackGemm ? nl * 4 + (lgrp ^ ((nl >> 1) & 3))
                                          : (nl >> 4) * 64 + lgrp * 16 + (nl & 15);
      woff[f] = oc(f) < g.Cout ? tile * ca.wtile + in * 16 : kOutOfRange;
    }
  };

  // the outputs of the unfinished pass: pixel m of the first R outputs'
  // stands for that pixel of the unfinished output in the same slot
  auto open_output = [&](int tau) { return tail_output(ca.E, ca.R, ca.fd_R, tau); };
  auto continues = [&](int t0) { return continues_sum(ca.n0, g.kT, g.dT, ca.fd_dT, t0); };

  // a copy the compiler cannot trace: the pixel arithmetic of the prologue and
  // the epilogue is the same in both passes, and kept in registers across the
  // K loop it would spill
  auto fresh = [](int v) {
    __asm__ volatile("" : "+s"(v));
    return v;
  };

  for (int pass = 0; pass < 2; ++pass) {
    if (pass == 0 && m0 >= ca.E * ca.So) continue;  // (uniform)
    if (pass == 1 && (!ca.tail || m0 >= ca.R * ca.So)) break;

    const int first = pass == 0 ? fdiv(max(m0, 0), ca.fd_So) : ca.E;  // lowest output of the tile
    // temporal taps that fall on a frame of the call for some output of the tile
    const int last = pass == 0 ? fdiv(min(m0 + M_WG, ca.E * ca.So) - 1, ca.fd_So) : ca.nu - 1;
    const int tlo = first * g.sT + ca.c0, thi = last * g.sT + ca.c0;
    const int j_lo = thi < 0 ? (-thi + g.dT - 1) / g.dT : 0;
    const int j_hi = ca.T - 1 - tlo < 0 ? -1 : min(g.kT - 1, (ca.T - 1 - tlo) / g.dT);
    const int total = max(0, (j_hi - j_lo + 1) * ca.nq);

    if constexpr (WINDOW) {
      if (pass == 0 && total > 0) {
        // all the pixels that the tile's taps reach, with all their channels:
        // row r is pixel q0 + r of the planes
        const int rows = ca.win_rows, nrb = rows >> 7, CSn = ca.nq;
        const int q0 = ca.c0 * ca.S + m0;
        constexpr int NB = 3;  // row blocks whose loads are in flight together
        for (int i0 = 0; i0 < CSn * nrb; i0 += NB) {
          uint32_t wraw[NB][8];
          int sh[NB];
#pragma unroll
          for (int n = 0; n < NB; ++n) {
            const int i = i0 + n;
            const int cb = fdiv(i, ca.fd_nrb), rb = i - cb * nrb;
            const int qa = q0 + rb * 128 + 2 * lane;
            // where a pair reaches over the end of the planes, load the pair
            // beside it (a plane has two pixels at least)
            sh[n] = qa < 0 ? 1 : qa == ca.span - 1 ? -1 : 0;
            const bool in = (qa >= -1) & (qa < ca.span) & (i < CSn * nrb);
            uint32_t vo = in ? uint32_t((qa + sh[n]) + (cb * 32 + wave * 8) * ca.plane) * 2u
                             : uint32_t(kOutOfRange);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              wraw[n][e] = __builtin_amdgcn_raw_buffer_load_b32(xr, int(vo), 0, 0);
              vo += uint32_t(ca.plane) * 2u;
            }
          }
#pragma unroll
          for (int n = 0; n < NB; ++n) {
            const int i = i0 + n;
            if (i >= CSn * nrb) break;  // uniform
            const int cb = fdiv(i, ca.fd_nrb), rb = i - cb * nrb;
            uint32_t(&r)[8] = wraw[n];
            if (__any(sh[n])) {  // uniform: at the clip's ends
#pragma unroll
              for (int e = 0; e < 8; ++e)
                r[e] = sh[n] > 0 ? r[e] << 16 : sh[n] < 0 ? r[e] >> 16 : r[e];
            }
            uint4 u0, u1;
            pair_units(r, u0, u1);
            const int row = rb * 128 + 2 * lane;
            uint4* at = clip_lds + (cb * rows + row) * 4 + (wave ^ ((row >> 1) & 3));
            at[0] = u0;
            at[4] = u1;
          }
        }
      }
    }

    // ---- the pixels this lane stages -----------------------------------
    // element offset of tap (0, 0, 0) in channel 0, its call frame and its
    // row and column (both may lie outside)
    int base[NBLK], fr[NBLK][PAIR ? 2 : 1], hw[NBLK];
#pragma unroll
    for (int i = 0; i < NBLK; ++i) {
      const int blk = ((i * NW + wave) >> 2) % MB;
#pragma unroll
      for (int h = 0; h < (PAIR ? 2 : 1); ++h) {
        const int m = m0 + blk * PXB + (PAIR ? 2 * lane + h : lane);
        const int tau = fdiv(max(m, 0), ca.fd_So), p = m - tau * ca.So;
        int to = tau;
        bool in = m >= 0;
        if (pass == 1) {  // uniform
          to = open_output(tau);
          in = in & (tau < ca.R) & (to < ca.nu);
        }
        const int t0 = to * g.sT + ca.c0;
        fr[i][h] = in ? t0 : kNoFrame;
        const int io = fdiv(p, ca.fd_Wo), jo = p - io * g.Wo;
        const int hi = io * g.sH - g.pH, wi = jo * g.sW - g.pW;
        if (!PAIR) hw[i] = ca.unpadded ? 0 : (hi << 16) | (wi & 0xffff);
        // (of a pair, the first pixel's, or where that has no output the
        // second's less one)
        if (h == 0 || fr[i][0] == kNoFrame) base[i] = t0 * ca.S + hi * g.W + wi - h;
      }
    }

    // ---- accumulators ------------------------------------------------------
    v4f acc[WMF][WNF];
#pragma unroll
    for (int mf = 0; mf < WMF; ++mf)
#pragma unroll
      for (int f = 0; f < WNF; ++f) acc[mf][f] = v4f{0.f, 0.f, 0.f, 0.f};
    if (first * g.sT + ca.c0 < 0 && ca.n0 > 0) {  // uniform: some may continue
      const int m0h = fresh(m0);
#pragma unroll
      for (int mf = 0; mf < WMF; ++mf)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = m0h + wm * (16 * WMF) + mf * 16 + lgrp * 4 + r;
          const int tau = fdiv(max(m, 0), ca.fd_So), p = m - tau * ca.So;
          const int to = pass == 0 ? tau : open_output(tau);
          const bool in = (m >= 0) & (pass == 0 ? to < ca.E : (tau < ca.R) & (to < ca.nu)) &
                          continues(to * g.sT + ca.c0);
          const int s = ca.slot0 + to;
          const int off = (s - fdiv(s, ca.fd_R) * ca.R) * ca.ring_slot + b * ca.So + p;
#pragma unroll
          for (int f = 0; f < WNF; ++f)
            acc[mf][f][r] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(
                rr, in & (oc(f) < g.Cout) ? (off + oc(f) * g.B * ca.So) * 4 : kOutOfRange, 0, 0));
          __builtin_amdgcn_sched_barrier(0);
        }
    }

    // ---- K loop ------------------------------------------------------------
    // The gathers run through the tile's k-steps in order: temporal tap j,
    // then (a, c) over spatial taps and channel blocks in the step kernel's
    // nesting.  A k-step's lane offsets change only with its taps.  Every load
    // of the loop issues unconditionally (k-steps past the last and pixels
    // outside read out of range), so that the compiler's count of requests in
    // flight stays exact and a stage waits for its own operands only.
    constexpr int RL = KL;                      // raw loads per item
    struct Walk {
      int j, a, c;
      int key;  // the taps voff holds
    };
    Walk wk{j_lo, 0, 0, -1};
    int voff[NBLK];
    int mode[NBLK];        // PAIR: 1, -1 where the pair's load was moved by one pixel
    uint64_t moved[NBLK];  // the lanes where it was
    uint32_t raw[PD][ITEMS][RL];
    int rmode[PD][NBLK];
    uint64_t rmoved[PD][NBLK];
    const int lim_c = int(ca.fd_q.d), lim_a = ca.nq / lim_c;
    auto forward = [&]() __attribute__((always_inline)) {
      if (++wk.c == lim_c) {
        wk.c = 0;
        if (++wk.a == lim_a) {
          wk.a = 0;
          ++wk.j;
        }
      }
    };
    auto locate = [&]() __attribute__((always_inline)) {
      const int sp = ca.tap_outer ? wk.a : wk.c;
      const int key = wk.j * ca.ntaps + sp;
      if (key == wk.key) return;  // uniform
      wk.key = key;
      const int u = fdiv(sp, ca.fd_kW), v = sp - u * g.kW;
      const int dt = wk.j * g.dT;
      const int tap = dt * ca.S + u * g.dH * g.W + v * g.dW;
      const int frames = wk.j <= j_hi ? ca.T : 0;  // (none past the last k-step)
#pragma unroll
      for (int i = 0; i < NBLK; ++i) {
        if constexpr (PAIR) {
          const bool va = unsigned(fr[i][0] + dt) < unsigned(frames);
          const bool vb = unsigned(fr[i][1] + dt) < unsigned(frames);
          // where a pair reaches over the end of the planes, load the pair
          // beside it (a plane has two pixels at least)
          const int qa = base[i] + tap;
          const int sh = qa < 0 ? 1 : qa == ca.span - 1 ? -1 : 0;
          mode[i] = sh;
          moved[i] = __ballot((sh != 0) & (va | vb));
          voff[i] = (va | vb) ? (qa + sh) * esz : kOutOfRange;
        } else {
          const int hi = (hw[i] >> 16) + u * g.dH, wi = int(int16_t(hw[i] & 0xffff)) + v * g.dW;
          const bool ok = (unsigned(fr[i][0] + dt) < unsigned(frames)) &
                          (unsigned(hi) < unsigned(g.H)) & (unsigned(wi) < unsigned(g.W));
          voff[i] = ok ? (base[i] + tap) * esz : kOutOfRange;
        }
      }
    };
    // the next stage's gathers, into raw slot `slot`
    auto load_a = [&](int slot) __attribute__((always_inline)) {
      locate();
      if constexpr (PAIR) {
#pragma unroll
        for (int i = 0; i < NBLK; ++i) {
          rmode[slot][i] = mode[i];
          rmoved[slot][i] = moved[i];
        }
      }
#pragma unroll
      for (int it = 0; it < ITEMS; ++it) {
        const int idx = it * NW + wave;
        const int i = NBLK == 1 ? 0 : it % NBLK;
        const int ch = (ca.tap_outer ? wk.c : wk.a) * CK + (idx & 3) * ca.cgrp;
        if constexpr (FAR) {
          uint32_t co = min(uint32_t(min(ch, g.Cin) * ca.plane) * uint32_t(esz),
                            uint32_t(x_bytes));
#pragma unroll
          for (int e = 0; e < RL; ++e) {
            if constexpr (esz == 4)
              raw[slot][it][e] = __builtin_amdgcn_raw_buffer_load_b32(xr, voff[i], int(co), 0);
            else
              raw[slot][it][e] = __builtin_amdgcn_raw_buffer_load_b16(xr, voff[i], int(co), 0);
            co = min(co + ca.celt, uint32_t(x_bytes));
          }
        } else {
          uint32_t vo = uint32_t(voff[i]) + uint32_t(ch * ca.plane * esz);
#pragma unroll
          for (int e = 0; e < RL; ++e) {
            if constexpr (esz == 4 || PAIR)
              raw[slot][it][e] = __builtin_amdgcn_raw_buffer_load_b32(xr, int(vo), 0, 0);
            else
              raw[slot][it][e] = __builtin_amdgcn_raw_buffer_load_b16(xr, int(vo), 0, 0);
            vo += ca.celt;
          }
        }
      }
      forward();
    };
    auto store_a = [&](int slot, int buf) __attribute__((always_inline)) {
#pragma unroll
      for (int it = 0; it < ITEMS; ++it) {
        const int idx = it * NW + wave;
        const int grp = idx & 3, blk = (idx >> 2) % MB;
        auto put = [&](int px, const uint4& u) { As[buf][px * 4 + (grp ^ ((px >> 1) & 3))] = u; };
        uint32_t(&r)[RL] = raw[slot][it];
        if constexpr (esz == 4) {
          put(blk * PXB + lane, make_uint4(r[0], r[1], r[2], r[3]));
        } else if constexpr (PAIR) {
          const int i = NBLK == 1 ? 0 : it % NBLK;
          const int md = rmode[slot][i];
          if (rmoved[slot][i]) {  // uniform: at the clip's ends
#pragma unroll
            for (int e = 0; e < RL; ++e)
              r[e] = md > 0 ? r[e] << 16 : md < 0 ? r[e] >> 16 : r[e];
          }
          uint4 u0, u1;
          pair_units(r, u0, u1);
          put(blk * PXB + 2 * lane, u0);
          put(blk * PXB + 2 * lane + 1, u1);
        } else {
          put(blk * PXB + lane, make_uint4(r[0] | (r[1] << 16), r[2] | (r[3] << 16),
                                           r[4] | (r[5] << 16), r[6] | (r[7] << 16)));
        }
      }
    };
    Frag bq[2][WNF];
    // the weights' walk: k-step within the tap, its offset, k-steps left (past
    // the last one the weights are zero, as the pixels are)
    int bj = j_lo, bk = 0, bso = 0, bleft = total;
    weight_cols(bj);
    auto load_b = [&](int slot) __attribute__((always_inline)) {
      // (the bounds check takes the scalar offset from the size: none on an
      // empty buffer)
      const __amdgpu_buffer_rsrc_t wr = make_rsrc(wp, bleft > 0 ? ca.w_bytes : 0);
      const int so = bleft > 0 ? bso : 0;
#pragma unroll
      for (int f = 0; f < WNF; ++f)
        bq[slot][f] = __builtin_bit_cast(
            Frag, __builtin_amdgcn_raw_buffer_load_b128(wr, woff[f], so, 0));
      --bleft;
      bso += ca.wq;
      if (++bk == ca.nq) {  // uniform, no memory request inside
        bk = 0;
        if (ca.tap_cols == 0) {
          bso += ca.tap_bytes;  // to k-step 0 of the next tap
        } else {
          bso = 0;
          weight_cols(++bj);
        }
      }
    };
    // a k-step's pixel operands are requested four fragments at a time, the
    // first ones before the next stage's gathers
    Frag af[4];
    auto operands = [&](int buf, int h) __attribute__((always_inline)) {
#pragma unroll
      for (int mf = 0; mf < 4; ++mf) {
        const int px = wm * (16 * WMF) + (h + mf) * 16 + lrow;
        af[mf] = __builtin_bit_cast(Frag, As[buf][px * 4 + (lgrp ^ ((px >> 1) & 3))]);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    auto multiply = [&](int buf, int slot) __attribute__((always_inline)) {
#pragma unroll
      for (int h = 0; h < WMF; h += 4) {
        if (h > 0) operands(buf, h);
        // (fp32: a unit's four k-steps of one accumulator lie 4 * WNF
        // instructions apart)
#pragma unroll
        for (int i = 0; i < (esz == 4 ? 4 : 1); ++i)
#pragma unroll
          for (int mf = 0; mf < 4; ++mf)
#pragma unroll
            for (int f = 0; f < WNF; ++f) clip_mma(acc[h + mf][f], af[mf], bq[slot][f], i);
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    bool staged = false;
    if constexpr (WINDOW) {
      if (pass == 0 && total > 0) {
        staged = true;
        const int rows = ca.win_rows, CSn = ca.nq;
        load_b(0);
        __syncthreads();
        // the tile's k-steps, without a barrier
        Frag wf[4];
        int aj = j_lo, ac = 0;
        const uint4* at = nullptr;
        auto window_row = [&]() __attribute__((always_inline)) {
          const int row = wm * (16 * WMF) + lrow + aj * g.dT * ca.S;
          at = clip_lds + row * 4 + (lgrp ^ ((row >> 1) & 3));
        };
        window_row();
        auto window_operands = [&](int h) __attribute__((always_inline)) {
#pragma unroll
          for (int mf = 0; mf < 4; ++mf) wf[mf] = __builtin_bit_cast(Frag, at[(h + mf) * 64]);
          __builtin_amdgcn_sched_barrier(0);
        };
        auto window_next = [&]() __attribute__((always_inline)) {
          at += rows * 4;
          if (++ac == CSn) {  // uniform
            ac = 0;
            // (past the last tap the reads repeat its rows, unused)
            if (aj < j_hi) ++aj;
            window_row();
          }
        };
        for (int k = 0;; k += 2) {
          bool done = false;
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            window_operands(0);
            load_b((i + 1) & 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int h = 0; h < WMF; h += 4) {
              if (h > 0) window_operands(h);
#pragma unroll
              for (int mf = 0; mf < 4; ++mf)
#pragma unroll
                for (int f = 0; f < WNF; ++f) clip_mma(acc[h + mf][f], wf[mf], bq[i][f], 0);
              __builtin_amdgcn_sched_barrier(0);
            }
            window_next();
            if (k + i + 1 >= total) {  // uniform
              done = true;
              break;
            }
          }
          if (done) break;
        }
        __syncthreads();  // the second pass stages into the same LDS
      }
    }
    if (!staged && total > 0) {
      load_b(0);
#pragma unroll
      for (int p = 0; p < PD; ++p) load_a(p);
      store_a(0, 0);
      __syncthreads();
      for (int st = 0;; st += UN) {
        bool done = false;
#pragma unroll
        for (int i = 0; i < UN; ++i) {
          operands(i & 1, 0);
          // requests complete in order: the weights, needed first, go first
          load_b((i + 1) & 1);
          load_a(i % PD);
          __builtin_amdgcn_sched_barrier(0);
          multiply(i & 1, i & 1);
          __builtin_amdgcn_sched_barrier(0);
          store_a((i + 1) % PD, (i + 1) & 1);
          __syncthreads();
          if (st + i + 1 >= total) {  // uniform
            done = true;
            break;
          }
        }
        if (done) break;
      }
    }

    // ---- epilogue ----------------------------------------------------------
    // lane (lrow, lgrp) of fragment (mf, f) holds channel oc(f) of the four
    // consecutive pixels m .. m + 3, consecutive in y too
    const int m0e = fresh(m0);
    if (pass == 0) {
      float bo[WNF];
#pragma unroll
      for (int f = 0; f < WNF; ++f)
        bo[f] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(br, oc(f) * 4, 0, 0));
      int row[WNF];  // byte offset of this lane's channels' first pixel in the tile
#pragma unroll
      for (int f = 0; f < WNF; ++f) {
        const uint32_t e = uint32_t(b * g.Cout + oc(f)) * uint32_t(ca.y_bc) +
                           uint32_t(m0e + wm * (16 * WMF) + lgrp * 4);
        row[f] = oc(f) < g.Cout ? int(e * uint32_t(esz)) : kOutOfRange;
#pragma unroll
        for (int mf = 0; mf < WMF; ++mf) acc[mf][f] += v4f{bo[f], bo[f], bo[f], bo[f]};
      }
      // (ReLU before the rounding, which keeps signs and order, is ReLU after it)
      if (ca.act == CO_ACT_RELU) {
#pragma unroll
        for (int mf = 0; mf < WMF; ++mf)
#pragma unroll
          for (int f = 0; f < WNF; ++f)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[mf][f][r] = fmaxf(acc[mf][f][r], 0.f);
      }
      // a tile inside the outputs stores whole lanes
      const bool inside = (m0e >= 0) & (m0e + M_WG <= ca.E * ca.So);
#pragma unroll
      for (int mf = 0; mf < WMF; ++mf) {
        const int m = m0e + wm * (16 * WMF) + mf * 16 + lgrp * 4;
        const int left = ca.E * ca.So - m;  // pixels of this lane that exist
        const bool whole = inside | ((left >= 4) & (m >= 0));
#pragma unroll
        for (int f = 0; f < WNF; ++f) {
          const v4f v = acc[mf][f];
          const int off = whole ? row[f] + mf * 16 * esz : kOutOfRange;
          if constexpr (esz == 2) {
            typedef uint32_t v2u __attribute__((ext_vector_type(2)));
            typedef __bf16 v4b __attribute__((ext_vector_type(4)));
            __builtin_amdgcn_raw_buffer_store_b64(
                __builtin_bit_cast(v2u, __builtin_convertvector(v, v4b)), yr, off, 0, 0);
          } else {
            typedef uint32_t v4u __attribute__((ext_vector_type(4)));
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, v), yr, off, 0, 0);
          }
        }
        if (!inside && !whole) {  // (the tile's last lane, or its first)
#pragma unroll
          for (int f = 0; f < WNF; ++f)
#pragma unroll
            for (int r = 0; r < 4; ++r)
              store_at(yr, (r < left) & (m + r >= 0) ? row[f] + (mf * 16 + r) * esz : kOutOfRange,
                       0, from_f32<T>(acc[mf][f][r]));
        }
      }
    } else {
#pragma unroll
      for (int mf = 0; mf < WMF; ++mf) {
        const int m = m0e + wm * (16 * WMF) + mf * 16 + lgrp * 4;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int tau = fdiv(max(m + r, 0), ca.fd_So), p = m + r - tau * ca.So;
          const int to = open_output(tau);
          const bool in = (m + r >= 0) & (tau < ca.R) & (to < ca.nu);
          const int s = ca.slot0 + to;
          const int off = (s - fdiv(s, ca.fd_R) * ca.R) * ca.ring_slot + b * ca.So + p;
#pragma unroll
          for (int f = 0; f < WNF; ++f)
            store_at(rr, in & (oc(f) < g.Cout) ? (off + oc(f) * g.B * ca.So) * 4 : kOutOfRange, 0,
                     acc[mf][f][r]);
        }
      }
    }
  }
}

struct ClipCall {
  const ConvGeom* g;
  const ConvLayout* L;
  char* state;
  const void* x;
  void* y;
  ClipArgs ca;
  hipStream_t s;
};

template <typename T, int WMF, int WNF, int NWM, int NWN, bool PAIR, bool WINDOW,
          bool FAR = false>
hipError_t clip_launch(ClipCall& c) {
  const ConvGeom& g = *c.g;
  ClipArgs& ca = c.ca;
  constexpr int M_WG = 16 * WMF * NWM, N_WG = 16 * WNF * NWN;
  const int64_t outputs = std::max<int64_t>(ca.E, ca.tail ? ca.R : 0);
  ca.m_pairs = int32_t(ceil_div(outputs * ca.So + ca.shift, M_WG) * g.B);
  ca.n_tiles = int32_t(ceil_div(g.Cout, N_WG));
  ca.fd_nt = make_fastdiv(uint32_t(ca.n_tiles));
  const int64_t blocks = ceil_div(ca.m_pairs, 8) * 8 * ca.n_tiles;
  if (blocks == 0) return hipSuccess;
  const size_t stages = size_t(2) * M_WG * 64;
  const size_t window = WINDOW ? size_t(ca.nq) * ca.win_rows * 64 : 0;
  auto kern = conv_clip_gemm_kernel<T, WMF, WNF, NWM, NWN, PAIR, WINDOW, FAR>;
  if constexpr (WINDOW) {
    const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                             hipFuncAttributeMaxDynamicSharedMemorySize,
                                             kClipWindowBytes);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kern, dim3(unsigned(blocks)),
                     dim3(64 * NWM * NWN), std::max(stages, window), c.s, g, ca, static_cast<const T*>(c.x),
                     static_cast<T*>(c.y), reinterpret_cast<const uint4*>(c.state + c.L->weight),
                     reinterpret_cast<const float*>(c.state + c.L->bias),
                     reinterpret_cast<float*>(c.state + c.L->ring));
  return hipGetLastError();
}

template <typename T, bool PAIR, bool WINDOW>
hipError_t clip_dispatch(ClipCall& c, int tile) {
  switch (tile) {
    case 32: return clip_launch<T, 4, 1, 2, 2, PAIR, WINDOW>(c);
    case 64: return clip_launch<T, 4, 2, 2, 2, PAIR, WINDOW>(c);
    case 96: return clip_launch<T, 4, 3, 2, 2, PAIR, WINDOW>(c);
    case 128: return clip_launch<T, 4, 4, 2, 2, PAIR, WINDOW>(c);
  }
  if constexpr (sizeof(T) == 2 && !PAIR) return clip_launch<T, 8, 3, 1, 4, PAIR, WINDOW>(c);
  return hipErrorInvalidValue;
}

}  // namespace

// Whether the clip GEMM takes a layer's buffers: GEMM-family weights whose
// step kernel folds each temporal tap in one chain (with the taps split over
// two waves, all of them in the first), 32-bit byte offsets everywhere.
bool clip_gemm_supported(const ConvGeom& g, int64_t x_frames, int64_t y_frames) {
  const int64_t lim = int64_t(1) << 31;
  const int64_t esz = g.dtype == CO_BF16 ? 2 : 4;
  if (g.algo == CO_ALGO_GEMM_REG) {
    RegConfig c;
    if (!reg_config(g, g.cfg, &c) || g.kH * g.kW > c.TAPS / c.KSPLIT) return false;
  } else if (g.algo != CO_ALGO_GEMM) {
    return false;
  }
  const ConvLayout L = conv_layout(g);
  return g.G == 1 &&
         (clip_unpadded(g) || (g.H < 16384 && g.W < 16384 && g.pH < 8192 && g.pW < 8192)) &&
         int64_t(g.B) * g.Cin * x_frames * g.S() * esz < lim &&
         int64_t(g.B) * g.Cout * y_frames * g.So() * esz < lim &&
         (x_frames + g.f) * g.So() < lim / 4 && int64_t(g.R) * L.ring_slot_elems * 4 < lim &&
         L.weight_bytes < lim;
}

hipError_t launch_conv_clip_gemm(const ConvGeom& g, const ConvLayout& L, char* state,
                                 const void* x, int64_t x_bc, int32_t nreal, int32_t count,
                                 void* y, int64_t y_bc, int64_t n0, bool update, int32_t act,
                                 hipStream_t s) {
  const int64_t esz = g.dtype == CO_BF16 ? 2 : 4;
  ClipCall c{&g, &L, state, x, y, ClipArgs{}, s};
  ClipArgs& ca = c.ca;
  static_cast<FrameSpan&>(ca) = frame_span(g, n0, nreal, count, update);
  ca.plane = int32_t(x_bc);
  ca.span = int32_t(int64_t(nreal) * g.S());
  ca.y_bc = int32_t(y_bc);
  ca.y_bytes = int32_t(int64_t(g.B) * g.Cout * y_bc * esz);
  ca.w_bytes = int32_t(L.weight_bytes);
  ca.ring_slot = int32_t(L.ring_slot_elems);
  ca.ring_bytes = int32_t(int64_t(g.R) * L.ring_slot_elems * 4);
  const int KL = g.dtype == CO_BF16 ? 8 : 4;
  const int ntaps = g.kH * g.kW;
  const int CS = int(ceil_div(g.Cin, 4 * KL));
  ca.ntaps = ntaps;
  ca.nq = ntaps * CS;
  ca.cgrp = KL;
  const int64_t lim = int64_t(1) << 31;
  ca.celt = uint32_t(x_bc * esz);  // (below 2^31, as C_in planes are)
  if (g.algo == CO_ALGO_GEMM_REG) {
    ca.pack = kPackReg;
    ca.tap_outer = 1;
    ca.wcols = 16;
    ca.wq = 1024;
    ca.wtile = ca.nq * 1024;
    if (g.dtype == CO_F32) {  // word e of lane group q holds channel 4 e + q
      ca.cgrp = 1;
      ca.celt = uint32_t(std::min(4 * x_bc * esz, lim));
    }
  } else {
    GemmConfig gc;
    if (!gemm_config(g, g.cfg, &gc)) return hipErrorInvalidValue;
    ca.pack = gc.ws ? kPackWs : kPackGemm;
    ca.tap_outer = 0;
    ca.wcols = gc.N_WG;
    ca.wq = gc.N_WG * 64;
    ca.wtile = ca.nq * ca.wq;
  }
  ca.tap_cols = g.Cout % ca.wcols;
  ca.tap_bytes = int32_t(int64_t(g.Cout / ca.wcols) * ca.wtile - int64_t(ca.nq) * ca.wq);
  ca.act = act;
  ca.unpadded = clip_unpadded(g);
  ca.fd_B = make_fastdiv(uint32_t(g.B));
  ca.fd_So = make_fastdiv(uint32_t(ca.So));
  ca.fd_Wo = make_fastdiv(uint32_t(g.Wo));
  ca.fd_R = make_fastdiv(uint32_t(g.R));
  ca.fd_dT = make_fastdiv(uint32_t(g.dT));
  ca.fd_q = make_fastdiv(uint32_t(ca.tap_outer ? CS : ntaps));
  ca.fd_kW = make_fastdiv(uint32_t(g.kW));
  ca.fd_wcols = make_fastdiv(uint32_t(ca.wcols));
  const int tile = clip_tile(g, ca.E);
  // Where a channel of the last k-step has no 32-bit offset from kOutOfRange
  // (few channels, long clips): any tile gives the same bits, one is built.
  const bool far = round_up(g.Cin, 4 * KL) * x_bc * esz > lim;
  if (g.dtype == CO_F32)
    return far ? clip_launch<float, 4, 2, 2, 2, false, false, true>(c)
               : clip_dispatch<float, false, false>(c, tile);
  if (far) return clip_launch<bf16_t, 4, 2, 2, 2, false, false, true>(c);
  if (!clip_pairs(g) || ca.span < 2) return clip_dispatch<bf16_t, false, false>(c, tile);
  // slots wrap around to output E at the pixel (E mod R) So of a tile row
  ca.shift = ca.tail ? int32_t((int64_t(ca.E % g.R) * ca.So) & 1) : 0;
  // the tile's pixels and those its later taps add, in LDS at once
  const int64_t rows = round_up(128 + int64_t(g.kT - 1) * g.dT * ca.S, 128);
  if (g.kT > 1 && rows * ca.nq * 64 <= kClipWindowBytes) {
    ca.win_rows = int32_t(rows);
    ca.fd_nrb = make_fastdiv(uint32_t(rows / 128));
    return clip_dispatch<bf16_t, true, true>(c, tile);
  }
  return clip_dispatch<bf16_t, true, false>(c, tile);
}

}  // namespace coinf
