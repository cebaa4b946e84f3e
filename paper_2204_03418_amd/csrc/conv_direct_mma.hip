// Matrix-core convolution of ungrouped direct layers: strided or dilated
// planes, taps and channel counts that no packed GEMM layout holds.  One
// kernel serves the eager step (a buffer of one frame) and forward_steps, so
// stepping and buffers give the same bits.
//
// Implicit GEMM over a call's frames: rows are the output pixels of one
// stream, all its frames in a row (m = frame * Ho * Wo + pixel, the order of
// y), columns the output channels, depth (temporal tap, then k = the flat
// index of (channel, u, v)), in k-steps of 32 (bf16 weights) or 16.  Outputs
// begin with their partial sum in the ring where a tap came before the call,
// and end in the ring where the call does not complete them.
//
// The weights stay as the direct layout keeps them, float32 in the caller's
// order (o, c, j, u, v): a k-step's are gathered along k, where a temporal
// tap's kH kW values lie side by side, and staged in LDS in operand order.
// Both operands of a k-step are requested one k-step ahead in registers and
// double buffered in LDS.  Input taps outside the plane or the call are
// addressed out of range (zero): a pixel keeps one bit per spatial tap, which
// becomes the sign of its byte offset.
//
// Arithmetic.  bf16 frames with the bf16 weights the caller gave (exact in
// the top halves of the float32 ones) use the bf16 matrix instructions, whose
// products are exact; float32 frames, and bf16 frames with weights that a
// batch normalisation was folded into, the float32 ones.  Sums are float32.
//
// What bounds it: the gathers, 2 or 4 bytes a lane, through the CUs' address
// and L1 pipes: 112 wave loads for a k-step of 128 pixels x 96 channels, about
// 1000 of its 1200 cycles at three workgroups a CU, where the matrix
// instructions take 200.  192-channel tiles halve the pixels' share but leave
// two workgroups a CU (321 us against 277 when both were built; the kernel took
// 253 us after that, in the first measure below).
//
// Measured against a thread per output and a launch per frame: 96 -> 192,
// 3x3x3, spatial stride 2, 28x28, 16 streams, bf16: 16 frames 12.2 ms -> 253
// us, a step 764 -> 74 us; float32, 4 streams, 16 frames 4.6 ms -> 295 us;
// 1x3x3, 128 -> 256, 4 streams 5.1 ms -> 70 us.
#include <algorithm>
#include <type_traits>

#include "device.hpp"
#include "launch.hpp"

namespace coinf {

namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef __bf16 v8bf __attribute__((ext_vector_type(8)));

// A call frame that no tap moves into the call.
constexpr int kNoFrame = -(1 << 29);

struct DmArgs : FrameSpan {
  int32_t m_pairs, n_tiles;  // (pixel tile, stream) pairs; channel tiles
  int32_t plane, x_bytes;    // elements between input channels; a stream's bytes
  int32_t y_bc, y_bytes;     // elements between output channels; a stream's bytes
  int32_t w_bytes, ring_bytes, ring_slot;
  int32_t kt, nq;    // k values and k-steps of a temporal tap
  int32_t khw;       // spatial taps
  int64_t x_plane, y_plane;  // FAR: elements between input and output channels
  FastDiv fd_nt, fd_B, fd_So, fd_Wo, fd_R, fd_khw, fd_kW, fd_dT;
};

// BF: bf16 matrix instructions (else float32).  MB: 64-pixel blocks of the
// workgroup's tile; 2 x 2 waves of 32 MB pixels x 16 WNF channels.  FAR: one
// frame whose planes lie past 32-bit offsets of each other (a step on a frame
// of a large buffer): every channel has a resource of its own.
template <typename T, bool BF, int MB, int WNF, bool FAR>
__global__ __launch_bounds__(256, MB * WNF > 6 ? 2 : 3) void conv_direct_mma_kernel(
    ConvGeom g, DmArgs ca, const T* __restrict__ x, int64_t x_stream, T* __restrict__ y,
    int64_t y_stream, const float* __restrict__ w, const float* __restrict__ bias,
    float* __restrict__ ring) {
  constexpr int esz = int(sizeof(T));
  constexpr int KL = BF ? 8 : 4;    // k values per 16-byte unit
  constexpr int CK = 4 * KL;        // k values per k-step
  constexpr int WMF = 2 * MB;       // 16-pixel fragments per wave
  constexpr int M_WG = 64 * MB, N_WG = 32 * WNF;
  constexpr int CPL = 64 / CK;      // channels of one wave's weight load
  constexpr int NL = N_WG / (4 * CPL);  // weight loads per lane and k-step
  using Frag = typename std::conditional<BF, v8bf, v4f>::type;
  __shared__ uint4 As[2][M_WG * 4];
  __shared__ uint4 Bs[2][N_WG * 4];

  const int tid = int(threadIdx.x);
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lrow = lane & 15, lgrp = lane >> 4;
  const int wm = wave >> 1, wn = wave & 1;

  // Blocks are dealt to the 8 XCDs in turn: the channel tiles of one pixel
  // tile run on one XCD, one after the other, and share its input in L2.
  const int bid = int(blockIdx.x) >> 3;
  const int bp = fdiv(bid, ca.fd_nt);
  const int nt = bid - bp * ca.n_tiles;
  const int pair = bp * 8 + (int(blockIdx.x) & 7);
  if (pair >= ca.m_pairs) return;  // whole workgroups
  const int mt = fdiv(pair, ca.fd_B), b = pair - mt * g.B;
  const int m0 = mt * M_WG;

  const T* xb = x + b * x_stream;
  const __amdgpu_buffer_rsrc_t xr = make_rsrc(xb, ca.x_bytes);
  const __amdgpu_buffer_rsrc_t yr = make_rsrc(y + b * y_stream, ca.y_bytes);
  const __amdgpu_buffer_rsrc_t rr = make_rsrc(ring, ca.ring_bytes);
  const __amdgpu_buffer_rsrc_t wr = make_rsrc(w, ca.w_bytes);
  const __amdgpu_buffer_rsrc_t br = make_rsrc(bias, g.Cout * 4);

  // this lane's output channel in fragment f
  auto oc = [&](int f) { return nt * N_WG + (wn * WNF + f) * 16 + lrow; };
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

    // the outputs of the tile, and the temporal taps that fall on a frame of
    // the call for some of them
    int first = fdiv(m0, ca.fd_So);
    int last = fdiv(min(m0 + M_WG, (pass == 0 ? ca.E : ca.R) * ca.So) - 1, ca.fd_So);
    if (pass == 1) {
      if (last - first < 4) {
        int lo = ca.nu, hi = -1;
        for (int tau = first; tau <= last; ++tau) {
          const int to = open_output(tau);
          if (to < ca.nu) {
            lo = min(lo, to);
            hi = max(hi, to);
          }
        }
        if (hi < 0) break;  // slots without an unfinished output
        first = lo;
        last = hi;
      } else {
        first = ca.E;
        last = ca.nu - 1;
      }
    }
    const int tlo = first * g.sT + ca.c0, thi = last * g.sT + ca.c0;
    const int j_lo = thi < 0 ? fdiv(-thi + g.dT - 1, ca.fd_dT) : 0;
    const int j_hi = ca.T - 1 - tlo < 0 ? -1 : min(g.kT - 1, fdiv(ca.T - 1 - tlo, ca.fd_dT));
    const int total = max(0, (j_hi - j_lo + 1) * ca.nq);

    // ---- the pixels this lane stages -----------------------------------
    // byte offset of tap (j_lo, 0, 0) in channel 0 and its call frame; one bit
    // per spatial tap that lies outside the plane, and bit 31
    int base[MB], fr[MB];
    uint32_t outside[MB], nm[MB];
#pragma unroll
    for (int i = 0; i < MB; ++i) {
      const int m = m0 + i * 64 + lane;
      const int tau = fdiv(m, ca.fd_So), p = m - tau * ca.So;
      const int to = pass == 0 ? tau : open_output(tau);
      const bool in = pass == 0 ? tau < ca.E : (tau < ca.R) & (to < ca.nu);
      const int t0 = to * g.sT + ca.c0 + j_lo * g.dT;
      fr[i] = in ? t0 : kNoFrame;
      const int io = fdiv(p, ca.fd_Wo), jo = p - io * g.Wo;
      const int hi = io * g.sH - g.pH, wi = jo * g.sW - g.pW;
      base[i] = (t0 * ca.S + hi * g.W + wi) * esz;
      uint32_t bits = 0x80000000u;
      int uv = 0;
      for (int u = 0; u < g.kH; ++u)
        for (int v = 0; v < g.kW; ++v, ++uv) {
          const bool ok = (unsigned(hi + u * g.dH) < unsigned(g.H)) &
                          (unsigned(wi + v * g.dW) < unsigned(g.W));
          bits |= uint32_t(!ok) << uv;
        }
      outside[i] = bits;
    }

    // ---- accumulators ------------------------------------------------------
    v4f acc[WMF][WNF];
#pragma unroll
    for (int mf = 0; mf < WMF; ++mf)
#pragma unroll
      for (int f = 0; f < WNF; ++f) acc[mf][f] = v4f{0.f, 0.f, 0.f, 0.f};
    if (tlo < 0 && ca.n0 > 0) {  // uniform: some may continue
      const int m0h = fresh(m0);
#pragma unroll
      for (int mf = 0; mf < WMF; ++mf)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int m = m0h + wm * (16 * WMF) + mf * 16 + lgrp * 4 + r;
          const int tau = fdiv(m, ca.fd_So), p = m - tau * ca.So;
          const int to = pass == 0 ? tau : open_output(tau);
          const bool in = (pass == 0 ? to < ca.E : (tau < ca.R) & (to < ca.nu)) &
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
    // Every load of the loop issues unconditionally (k-steps past the last
    // read out of range), so that the compiler's count of requests in flight
    // stays exact.
    uint32_t araw[MB][KL], braw[NL];
    int lj = j_lo, lq = 0;  // the next k-step to request
    auto tap = [&]() __attribute__((always_inline)) {
      const int frames = lj <= j_hi ? ca.T : 0;  // (none past the last k-step)
#pragma unroll
      for (int i = 0; i < MB; ++i)
        nm[i] = unsigned(fr[i]) < unsigned(frames) ? outside[i] : 0xffffffffu;
    };
    // this lane's weights: k value and channel within a wave's load
    const int wk = lane & (CK - 1), wsub = lane / CK;
    const uint32_t wrow = uint32_t(ca.kt * g.kT) * 4u;  // bytes between output channels
    const uint32_t wcol = uint32_t(nt * N_WG + wave * CPL + wsub) * wrow;
    auto load = [&]() __attribute__((always_inline)) {
      // weights first: the bf16 in a float32 is its upper half
      {
        const int k = lq * CK + wk;
        const int c = fdiv(k, ca.fd_khw);
        const bool in = (k < ca.kt) & (lj <= j_hi);
        uint32_t wo = in ? wcol + uint32_t(k + (c * (g.kT - 1) + lj) * ca.khw) * 4u
                         : uint32_t(kOutOfRange);
#pragma unroll
        for (int i = 0; i < NL; ++i) {
          if constexpr (BF)
            braw[i] = __builtin_amdgcn_raw_buffer_load_b16(wr, int(wo + 2u), 0, 0);
          else
            braw[i] = __builtin_amdgcn_raw_buffer_load_b32(wr, int(wo), 0, 0);
          wo += 4u * CPL * wrow;
        }
      }
      // the wave's k values of its unit: (c, u, v) of the first, then in order
      const int k0 = lq * CK + wave * KL;
      int c = fdiv(k0, ca.fd_khw);
      int uv = k0 - c * ca.khw;
      int u = fdiv(uv, ca.fd_kW), v = uv - u * g.kW;
#pragma unroll
      for (int e = 0; e < KL; ++e) {
        const bool in = k0 + e < ca.kt;
        const int chan = FAR ? 0 : c * ca.plane;
        const uint32_t off = in ? uint32_t(chan + u * g.dH * g.W + v * g.dW) * esz : 0u;
        const int sh = in ? 31 - uv : 0;
        const __amdgpu_buffer_rsrc_t cr =
            FAR ? make_rsrc(xb + (in ? c : 0) * ca.x_plane, ca.x_bytes) : xr;
#pragma unroll
        for (int i = 0; i < MB; ++i) {
          const uint32_t vo = ((nm[i] << sh) & 0x80000000u) | (uint32_t(base[i]) + off);
          if constexpr (esz == 2)
            araw[i][e] = __builtin_amdgcn_raw_buffer_load_b16(cr, int(vo), 0, 0);
          else
            araw[i][e] = __builtin_amdgcn_raw_buffer_load_b32(cr, int(vo), 0, 0);
        }
        ++uv;
        if (++v == g.kW) {
          v = 0;
          if (++u == g.kH) {
            u = 0;
            uv = 0;
            ++c;
          }
        }
      }
      if (++lq == ca.nq) {  // uniform, no memory request inside
        lq = 0;
        ++lj;
#pragma unroll
        for (int i = 0; i < MB; ++i) {
          fr[i] += g.dT;
          base[i] += g.dT * ca.S * esz;
        }
        tap();
      }
    };
    auto store = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int col = (i * 4 + wave) * CPL + wsub;
        const int grp = wk / KL;
        const int unit = (col >> 4) * 64 + grp * 16 + ((col & 15) ^ (grp << 2));
        if constexpr (BF)
          reinterpret_cast<uint16_t*>(Bs[buf])[unit * 8 + (wk & 7)] = uint16_t(braw[i]);
        else
          reinterpret_cast<uint32_t*>(Bs[buf])[unit * 4 + (wk & 3)] = braw[i];
      }
#pragma unroll
      for (int i = 0; i < MB; ++i) {
        const int px = i * 64 + lane;
        uint32_t(&r)[KL] = araw[i];
        uint4 v;
        if constexpr (BF)
          v = make_uint4(r[0] | (r[1] << 16), r[2] | (r[3] << 16), r[4] | (r[5] << 16),
                         r[6] | (r[7] << 16));
        else if constexpr (esz == 2)
          v = make_uint4(r[0] << 16, r[1] << 16, r[2] << 16, r[3] << 16);
        else
          v = make_uint4(r[0], r[1], r[2], r[3]);
        As[buf][px * 4 + (wave ^ ((px >> 1) & 3))] = v;
      }
    };
    auto multiply = [&](int buf, auto&& between) __attribute__((always_inline)) {
      Frag bq[WNF], af[WMF];
#pragma unroll
      for (int f = 0; f < WNF; ++f)
        bq[f] = __builtin_bit_cast(
            Frag, Bs[buf][(wn * WNF + f) * 64 + lgrp * 16 + (lrow ^ (lgrp << 2))]);
#pragma unroll
      for (int mf = 0; mf < WMF; ++mf) {
        const int px = wm * (16 * WMF) + mf * 16 + lrow;
        af[mf] = __builtin_bit_cast(Frag, As[buf][px * 4 + (lgrp ^ ((px >> 1) & 3))]);
      }
      __builtin_amdgcn_sched_barrier(0);
      between();
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (BF) {
#pragma unroll
        for (int mf = 0; mf < WMF; ++mf)
#pragma unroll
          for (int f = 0; f < WNF; ++f)
            acc[mf][f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[mf], bq[f], acc[mf][f], 0, 0, 0);
      } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int mf = 0; mf < WMF; ++mf)
#pragma unroll
            for (int f = 0; f < WNF; ++f)
              acc[mf][f] =
                  __builtin_amdgcn_mfma_f32_16x16x4f32(af[mf][i], bq[f][i], acc[mf][f], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    };
    if (total > 0) {
      tap();
      load();
      store(0);
      __syncthreads();
      for (int st = 0; st < total; ++st) {
        multiply(st & 1, load);
        store((st + 1) & 1);
        __syncthreads();
      }
    }

    // ---- epilogue ----------------------------------------------------------
    // lane (lrow, lgrp) of fragment (mf, f) holds channel oc(f) of the four
    // consecutive pixels m .. m + 3, consecutive in y too
    const int m0e = fresh(m0);
    if (pass == 0) {
      float bo[WNF];
      int row[WNF];  // byte offset of this lane's channels' first pixel in the tile
#pragma unroll
      for (int f = 0; f < WNF; ++f) {
        bo[f] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(br, oc(f) * 4, 0, 0));
        const uint32_t e =
            uint32_t(oc(f)) * uint32_t(ca.y_bc) + uint32_t(m0e + wm * (16 * WMF) + lgrp * 4);
        row[f] = oc(f) < g.Cout ? int(e * uint32_t(esz)) : kOutOfRange;
      }
#pragma unroll
      for (int mf = 0; mf < WMF; ++mf) {
        const int left = ca.E * ca.So - (m0e + wm * (16 * WMF) + mf * 16 + lgrp * 4);
        const bool whole = left >= 4;
#pragma unroll
        for (int f = 0; f < WNF; ++f) {
          const v4f v = acc[mf][f] + v4f{bo[f], bo[f], bo[f], bo[f]};
          if constexpr (FAR) {
            T* yo = y + b * y_stream + oc(f) * ca.y_plane + (ca.E * ca.So - left);
#pragma unroll
            for (int r = 0; r < 4; ++r)
              if (r < left && oc(f) < g.Cout) yo[r] = from_f32<T>(v[r]);
            continue;
          }
          const int off = whole && oc(f) < g.Cout ? row[f] + mf * 16 * esz : kOutOfRange;
          if constexpr (esz == 2) {
            typedef uint32_t v2u __attribute__((ext_vector_type(2)));
            typedef __bf16 v4b __attribute__((ext_vector_type(4)));
            __builtin_amdgcn_raw_buffer_store_b64(
                __builtin_bit_cast(v2u, __builtin_convertvector(v, v4b)), yr, off, 0, 0);
          } else {
            typedef uint32_t v4u __attribute__((ext_vector_type(4)));
            __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(v4u, v), yr, off, 0, 0);
          }
          if (!whole) {  // (the call's last lane)
#pragma unroll
            for (int r = 0; r < 3; ++r)
              store_at(yr, r < left && oc(f) < g.Cout ? row[f] + (mf * 16 + r) * esz : kOutOfRange,
                       0, from_f32<T>(v[r]));
          }
        }
      }
    } else {
#pragma unroll
      for (int mf = 0; mf < WMF; ++mf) {
        const int m = m0e + wm * (16 * WMF) + mf * 16 + lgrp * 4;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int tau = fdiv(m + r, ca.fd_So), p = m + r - tau * ca.So;
          const int to = open_output(tau);
          const bool in = (tau < ca.R) & (to < ca.nu);
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

// Pixel blocks of a tile: 128 pixels where those fill the CUs, else 64.
int dm_blocks(const ConvGeom& g, int64_t outputs, int n_tile) {
  const int64_t wgs = ceil_div(outputs * g.So(), 128) * g.B * ceil_div(g.Cout, n_tile);
  return wgs >= 256 ? 2 : 1;
}

// Channel tile: the least padded width times (1 + what staging a tile's input
// costs against its matrix work).
int dm_tile(const ConvGeom& g) {
  int best = 0;
  int64_t cost = 0;
  for (const int n : {64, 96, 128}) {
    const int64_t c = ceil_div(g.Cout, n) * (n + 32);
    if (best == 0 || c < cost) {
      best = n;
      cost = c;
    }
  }
  return best;
}

struct DmCall {
  const ConvGeom* g;
  const ConvLayout* L;
  char* state;
  const void* x;
  int64_t x_stream;
  void* y;
  int64_t y_stream;
  DmArgs ca;
  hipStream_t s;
};

template <typename T, bool BF, int MB, int WNF, bool FAR = false>
hipError_t dm_launch(DmCall& c) {
  const ConvGeom& g = *c.g;
  DmArgs& ca = c.ca;
  const int64_t outputs = std::max<int64_t>(ca.E, ca.tail ? ca.R : 0);
  ca.m_pairs = int32_t(ceil_div(outputs * ca.So, 64 * MB) * g.B);
  ca.n_tiles = int32_t(ceil_div(g.Cout, 32 * WNF));
  ca.fd_nt = make_fastdiv(uint32_t(ca.n_tiles));
  const int64_t blocks = ceil_div(ca.m_pairs, 8) * 8 * ca.n_tiles;
  if (blocks == 0) return hipSuccess;
  hipLaunchKernelGGL((conv_direct_mma_kernel<T, BF, MB, WNF, FAR>), dim3(unsigned(blocks)), dim3(256),
                     0, c.s, g, ca, static_cast<const T*>(c.x), c.x_stream, static_cast<T*>(c.y),
                     c.y_stream, reinterpret_cast<const float*>(c.state + c.L->weight),
                     reinterpret_cast<const float*>(c.state + c.L->bias),
                     reinterpret_cast<float*>(c.state + c.L->ring));
  return hipGetLastError();
}

template <typename T, bool BF>
hipError_t dm_dispatch(DmCall& c, bool far) {
  if (far) return dm_launch<T, BF, 1, 2, true>(c);  // (the same bits in any tile)
  const int tile = dm_tile(*c.g);
  const bool two = dm_blocks(*c.g, std::max<int64_t>(c.ca.E, c.ca.tail ? c.ca.R : 0), tile) == 2;
  switch (tile) {
    case 64: return two ? dm_launch<T, BF, 2, 2>(c) : dm_launch<T, BF, 1, 2>(c);
    case 96: return two ? dm_launch<T, BF, 2, 3>(c) : dm_launch<T, BF, 1, 3>(c);
    default: return two ? dm_launch<T, BF, 2, 4>(c) : dm_launch<T, BF, 1, 4>(c);
  }
}

}  // namespace

// Which layers: those whose taps hold 64 values or more, or 32 with a million
// multiplications a step.  Below, a step is a launch and a few k-steps either
// way (1 stream, 4 -> 16, 3x3x3, 4x4: 14.7 us on the direct kernel, 16.5 here;
// 64 -> 64, (3,), stride 2: 24.5 against 13; 8 -> 16, 1x3x3, 8x8: 15.8 against
// 12.2).
bool direct_mma_layer(const ConvGeom& g) {
  const int64_t khw = int64_t(g.kH) * g.kW;
  const int64_t macs = int64_t(g.B) * g.So() * g.Cout * g.Cin * khw * g.kT;
  // (a plain pointwise layer is direct only where it was asked for, and the
  // fused bottleneck step has its arithmetic)
  if (g.kT * khw == 1 && g.sT * g.sH * g.sW == 1) return false;
  return g.algo == CO_ALGO_DIRECT && g.G == 1 && g.Cout >= 16 && g.Cin * khw >= 32 && khw <= 31 &&
         (g.Cin * khw >= 64 || macs >= 1000000) && g.H < 16384 && g.W < 16384 && g.pH < 8192 &&
         g.pW < 8192 &&
         int64_t(g.R) * ring_slot_elems(g) * 4 < (int64_t(1) << 31) &&
         packed_weight_bytes(g) < (int64_t(1) << 28);
}

bool direct_mma_fits(const ConvGeom& g, int64_t x_bc, int64_t frames, int64_t y_bc) {
  const int64_t esz = g.dtype == CO_BF16 ? 2 : 4;
  return frames < (int64_t(1) << 24) && (g.Cin * x_bc + g.S()) * esz < 0x70000000 &&
         g.Cout * y_bc * esz < 0x70000000 && (frames + g.f) * g.So() < (int64_t(1) << 28);
}

bool direct_mma_step(const ConvGeom& g) {
  return direct_mma_layer(g) && direct_mma_fits(g, g.S(), 1, g.So());
}

hipError_t launch_direct_mma(const ConvGeom& g, const ConvLayout& L, char* state, const void* x,
                             int64_t x_bc, int32_t nreal, int32_t count, void* y, int64_t y_bc,
                             int64_t n0, bool update, hipStream_t s) {
  const int64_t esz = g.dtype == CO_BF16 ? 2 : 4;
  DmCall c{&g, &L, state, x, int64_t(g.Cin) * x_bc, y, int64_t(g.Cout) * y_bc, DmArgs{}, s};
  DmArgs& ca = c.ca;
  static_cast<FrameSpan&>(ca) = frame_span(g, n0, nreal, count, update);
  ca.plane = int32_t(x_bc);
  ca.x_bytes = int32_t((int64_t(g.Cin - 1) * x_bc + int64_t(nreal) * g.S()) * esz);
  ca.y_bc = int32_t(y_bc);
  ca.y_bytes = int32_t((int64_t(g.Cout - 1) * y_bc + int64_t(ca.E) * g.So()) * esz);
  ca.w_bytes = int32_t(L.weight_bytes);
  ca.ring_slot = int32_t(L.ring_slot_elems);
  ca.ring_bytes = int32_t(int64_t(g.R) * L.ring_slot_elems * 4);
  ca.khw = g.kH * g.kW;
  ca.kt = g.Cin * ca.khw;
  const bool bf = g.dtype == CO_BF16 && L.bf16_weights;
  ca.nq = int32_t(ceil_div(ca.kt, bf ? 32 : 16));
  ca.fd_B = make_fastdiv(uint32_t(g.B));
  ca.fd_So = make_fastdiv(uint32_t(ca.So));
  ca.fd_Wo = make_fastdiv(uint32_t(g.Wo));
  ca.fd_R = make_fastdiv(uint32_t(g.R));
  ca.fd_khw = make_fastdiv(uint32_t(ca.khw));
  ca.fd_kW = make_fastdiv(uint32_t(g.kW));
  ca.fd_dT = make_fastdiv(uint32_t(g.dT));
  const bool far = !direct_mma_fits(g, x_bc, nreal, y_bc);
  if (far) {  // one frame (launch_step_direct_mma)
    if (nreal != 1 || !direct_mma_step(g)) return hipErrorInvalidValue;
    ca.x_bytes = int32_t(g.S() * esz);
    ca.x_plane = x_bc;
    ca.y_plane = y_bc;
  }
  if (g.dtype == CO_F32) return dm_dispatch<float, false>(c, far);
  return bf ? dm_dispatch<bf16_t, true>(c, far) : dm_dispatch<bf16_t, false>(c, far);
}

hipError_t launch_step_direct_mma(const ConvGeom& g, const ConvLayout& L, char* state,
                                  const StepIO& io, const co_step_plan& plan, hipStream_t s) {
  // the step counter from a tap and the output it feeds; a plan without
  // unfinished outputs leaves the ring alone
  int64_t n0 = -1;
  bool update = false;
  for (int j = 0; j < plan.n_taps; ++j) {
    if (plan.action[j] == CO_TAP_NONE) continue;
    n0 = plan.target[j] * g.sT + int64_t(j) * g.dT - g.pT;
    update |= plan.action[j] == CO_TAP_START || plan.action[j] == CO_TAP_ACC;
  }
  if (n0 < 0) return hipSuccess;  // no tap
  return launch_direct_mma(g, L, state, io.x, io.x_bc, 1, 1, io.y, io.y_bc, n0, update, s);
}

}  // namespace coinf
