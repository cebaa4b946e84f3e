// Continual average / maximum pooling kernels.
//
// A pooling window factorises into a spatial reduction of each frame and a
// temporal reduction over the window's frames.  The state keeps the spatially
// reduced frames of the last f input frames in a FIFO of float32 frames
// (slot, B, C, Ho, Wo) plus one validity flag per slot (0 for end-padding
// frames).  Each step reduces the arriving frame once -- the intermediate
// result future outputs need, computed eagerly as section 3.1 describes
// before Principle 3 -- and, when the schedule emits, reduces the window's
// kT slots into the output.  Average pooling stores window sums (pads add 0)
// and divides once at emission; maximum pooling stores window maxima (pads
// are -inf).  Groups of lanes share each output element (see
// pool_step_kernel), so a window of 49 positions is loaded in one round.
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "device.hpp"
#include "launch.hpp"

namespace coinf {

namespace {

// Reduction of v over the G lanes of a lane group (G a power of two <= 64).
template <int G>
__device__ __forceinline__ float group_sum(float v) {
#pragma unroll
  for (int m = G / 2; m > 0; m >>= 1) v += __shfl_xor(v, m, G);
  return v;
}
template <int G>
__device__ __forceinline__ float group_max(float v) {
#pragma unroll
  for (int m = G / 2; m > 0; m >>= 1) v = fmaxf(v, __shfl_xor(v, m, G));
  return v;
}

// One pool step.  G lanes share one output element (b, c, i, j): they load
// the spatial window together (lane r takes window elements r, r + G, ...,
// with clamped addresses so all loads are in flight at once) and reduce it
// with cross-lane shuffles; the FIFO slot is written by lane 0; when the
// schedule emits, lane j of the group fetches temporal tap j and the group
// reduces again.  No thread ever waits on a chain of dependent loads.
template <typename T, int G>
__global__ __launch_bounds__(kBlock) void pool_step_kernel(
    PoolGeom g, const T* __restrict__ x, int64_t x_bc, T* __restrict__ y, int64_t y_bc,
    float* __restrict__ fifo, int64_t fifo_slot, float* __restrict__ valid, int32_t write_slot,
    int32_t update, int32_t emit, int32_t pad_frame, PoolTaps taps, FastDiv fd_So, FastDiv fd_Wo,
    FastDiv fd_kW) {
  const int32_t So = g.Ho * g.Wo;
  const int32_t total = g.B * g.C * So;
  const int64_t gid = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  const int32_t idx = int32_t(gid / G);  // output element of this lane's group
  const int32_t r = int32_t(gid % G);    // lane within the group
  const bool live = idx < total;         // whole groups are live or not
  const int32_t e_idx = live ? idx : 0;
  const int32_t bc = fdiv(e_idx, fd_So);
  const int32_t p = e_idx - bc * So;
  const int32_t i = fdiv(p, fd_Wo), jo = p - i * g.Wo;
  const bool is_max = g.kind == CO_POOL_MAX;
  const int32_t kHW = g.kH * g.kW;

  // spatial reduction of the arriving frame (out-of-frame positions read an
  // out-of-range buffer offset: zero, no branch around the load)
  float val = is_max ? -INFINITY : 0.f;
  const int x_extent =
      pad_frame ? 0 : int(((int64_t(g.B) * g.C - 1) * x_bc + g.H * g.W) * int64_t(sizeof(T)));
  const __amdgpu_buffer_rsrc_t xr = make_rsrc(x, x_extent);
  const int plane = int(int64_t(bc) * x_bc);
  for (int32_t e = r; e < kHW; e += G) {
    const int32_t u = fdiv(e, fd_kW), v = e - u * g.kW;
    const int32_t hi = i * g.sH + u * g.dH - g.pH;
    const int32_t wi = jo * g.sW + v * g.dW - g.pW;
    const bool in = hi >= 0 && hi < g.H && wi >= 0 && wi < g.W && !pad_frame;
    const float xv = load_or_zero<T>(xr, plane + hi * g.W + wi, in);
    if (in) val = is_max ? fmaxf(val, xv) : val + xv;
  }
  val = is_max ? group_max<G>(val) : group_sum<G>(val);
  if (!live) return;

  if (update && r == 0) {
    fifo[int64_t(write_slot) * fifo_slot + idx] = val;
    if (idx == 0) valid[write_slot] = pad_frame ? 0.f : 1.f;
  }
  if (!emit) return;

  // temporal reduction over the window's kT frames, spread over the group
  float acc = is_max ? -INFINITY : 0.f;
  float tcount = 0.f;
  for (int32_t t = r; t < g.kT; t += G) {
    const int32_t s = taps.src[t];
    if (s == -1) continue;  // start padding: ignored by max, adds 0 to a sum
    float ev, ok;
    if (s == -2) {          // the arriving frame
      ev = val;
      ok = pad_frame ? 0.f : 1.f;
    } else {
      ev = fifo[int64_t(s) * fifo_slot + idx];
      ok = valid[s];
    }
    acc = is_max ? fmaxf(acc, ev) : acc + ev;
    tcount += ok;
  }
  if (is_max) {
    acc = group_max<G>(acc);
  } else {
    acc = group_sum<G>(acc);
    tcount = group_sum<G>(tcount);
  }
  if (r != 0) return;
  float out;
  if (is_max) {
    out = acc;
  } else {
    // spatial positions inside the frame (count_include_pad = 0 divisor)
    int32_t vh = 0, vw = 0;
    for (int32_t u = 0; u < g.kH; ++u) {
      const int32_t hi = i * g.sH + u * g.dH - g.pH;
      vh += (hi >= 0 && hi < g.H) ? 1 : 0;
    }
    for (int32_t v = 0; v < g.kW; ++v) {
      const int32_t wi = jo * g.sW + v * g.dW - g.pW;
      vw += (wi >= 0 && wi < g.W) ? 1 : 0;
    }
    const float div = g.count_include_pad ? float(g.kT * kHW) : tcount * float(vh * vw);
    out = div > 0.f ? acc / div : 0.f;
  }
  y[int64_t(bc) * y_bc + p] = from_f32<T>(out);
}

template <typename T>
__global__ __launch_bounds__(kBlock) void pool_clip_kernel(PoolGeom g, int32_t T_in,
                                                           int32_t T_out,
                                                           const T* __restrict__ x,
                                                           T* __restrict__ y) {
  const int64_t So = int64_t(g.Ho) * g.Wo;
  const int64_t total = int64_t(g.B) * g.C * T_out * So;
  const int64_t idx = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  if (idx >= total) return;
  const int64_t p = idx % So;
  const int64_t t = (idx / So) % T_out;
  const int64_t bc = idx / (So * T_out);
  const int32_t i = int32_t(p / g.Wo), jo = int32_t(p % g.Wo);
  const int64_t S = int64_t(g.H) * g.W;
  const bool is_max = g.kind == CO_POOL_MAX;
  float acc = is_max ? -INFINITY : 0.f;
  int32_t count = 0;
  for (int32_t a = 0; a < g.kT; ++a) {
    const int64_t ti = t * g.sT + int64_t(a) * g.dT - g.pT;
    if (ti < 0 || ti >= T_in) continue;
    for (int32_t u = 0; u < g.kH; ++u) {
      const int32_t hi = i * g.sH + u * g.dH - g.pH;
      if (hi < 0 || hi >= g.H) continue;
      for (int32_t v = 0; v < g.kW; ++v) {
        const int32_t wi = jo * g.sW + v * g.dW - g.pW;
        if (wi < 0 || wi >= g.W) continue;
        const float e = to_f32<T>(x[(bc * T_in + ti) * S + hi * g.W + wi]);
        acc = is_max ? fmaxf(acc, e) : acc + e;
        ++count;
      }
    }
  }
  float out;
  if (is_max) {
    out = acc;
  } else {
    const int32_t div = g.count_include_pad ? g.kT * g.kH * g.kW : count;
    out = div > 0 ? acc / float(div) : 0.f;
  }
  y[idx] = from_f32<T>(out);
}

// ---- persistent forward_steps -------------------------------------------
//
// A clip of `count` frames in one launch (temporal stride 1 and dilation 1,
// a spatial window of at most G positions): the G lanes of output element
// (b, c, i, j) reduce each frame's window (one load per lane, the next
// frame's requested before the current one is reduced) and keep the last kT
// reduced frames and their validity in registers; when the schedule emits
// they reduce the window's frames into the output.  The FIFO is read at the
// start and written back at the end; the validity flags of the call's
// frames are written by the host afterwards.
struct PoolSteps {
  int64_t n0;     // step counter before the first frame
  int32_t count;  // frames: T real, then end padding
  int32_t T;
  int64_t emit0;  // first emitting step of the call: max(n0, d)
  int32_t sT;     // temporal stride: steps from n = d on emit every sT
  int32_t t_e0;   // first emitting frame of the call (count if none)
  int32_t update;
  int32_t x_bytes;  // bytes of the clip reachable from x
  int32_t y_bytes;  // bytes of the output clip
  int32_t fstride;  // bytes between consecutive frames
  FastDiv fd_So, fd_Wo, fd_kW;
};

template <typename T, int G, int KT, bool IS_MAX>
__global__ __launch_bounds__(kBlock) void pool_steps_kernel(
    PoolGeom g, PoolSteps ps, const T* __restrict__ x, int64_t x_bc, T* __restrict__ y,
    int64_t y_bc, float* __restrict__ fifo, int64_t fifo_slot, const float* __restrict__ valid) {
  const int32_t So = g.Ho * g.Wo;
  const int32_t total = g.B * g.C * So;
  const int64_t gid = int64_t(blockIdx.x) * kBlock + threadIdx.x;
  const int32_t idx = int32_t(gid / G);  // output element of this lane's group
  const int32_t r = int32_t(gid % G);    // lane within the group
  const bool live = idx < total;         // whole groups are live or not
  if (!live) return;                     // (no barrier follows)
  const int32_t bc = fdiv(idx, ps.fd_So);
  const int32_t p = idx - bc * So;
  const int32_t i = fdiv(p, ps.fd_Wo), jo = p - i * g.Wo;
  constexpr bool is_max = IS_MAX;  // (compile-time: no select per operation)
  const float neutral = is_max ? -INFINITY : 0.f;
  const int32_t kHW = g.kH * g.kW;

  // this lane's window position (at most one: kH*kW <= G)
  int32_t soff = -1;
  if (r < kHW) {
    const int32_t u = fdiv(r, ps.fd_kW), v = r - u * g.kW;
    const int32_t hi = i * g.sH + u * g.dH - g.pH;
    const int32_t wi = jo * g.sW + v * g.dW - g.pW;
    if (hi >= 0 && hi < g.H && wi >= 0 && wi < g.W) soff = hi * g.W + wi;
  }
  // divisor of an average with count_include_pad = 0: spatial positions in the frame
  int32_t vh = 0, vw = 0;
  for (int32_t u = 0; u < g.kH; ++u) {
    const int32_t hi = i * g.sH + u * g.dH - g.pH;
    vh += (hi >= 0 && hi < g.H) ? 1 : 0;
  }
  for (int32_t v = 0; v < g.kW; ++v) {
    const int32_t wi = jo * g.sW + v * g.dW - g.pW;
    vw += (wi >= 0 && wi < g.W) ? 1 : 0;
  }

  // fv[q], fok[q]: reduced value and validity of real frame n - (KT - 1) + q
  // at frame n; frames before the stream began are start padding
  float fv[KT], fok[KT];
#pragma unroll
  for (int q = 0; q + 1 < KT; ++q) {
    const int64_t rf = ps.n0 - (KT - 1) + q;
    const bool have = rf >= 0;
    fv[q] = have ? fifo[(rf % KT) * fifo_slot + idx] : neutral;
    fok[q] = have ? valid[rf % KT] : 0.f;
  }
  // the emitted value goes out through a buffer store that every lane issues
  // every frame, to the out-of-range offset unless lane 0 of a group emits:
  // a store under a branch would make the compiler wait for every frame in
  // flight before each frame
  const __amdgpu_buffer_rsrc_t yr = make_rsrc(y, ps.y_bytes);
  const int yoff = int((uint32_t(bc) * uint32_t(y_bc) + uint32_t(p)) * sizeof(T));
  // raw bits of this lane's window element of frame t (converted when the
  // frame is reduced, so the loads stay in flight); positions outside the
  // frame read the out-of-range offset and become the neutral value at use
  const __amdgpu_buffer_rsrc_t xr = make_rsrc(x, ps.x_bytes);
  const int loff = soff >= 0 ? int((uint32_t(bc) * uint32_t(x_bc) + uint32_t(soff)) * sizeof(T))
                             : kOutOfRange;
  // every frame issues its load (frames past the clip at the out-of-range
  // offset), so the compiler's count of loads in flight stays exact around
  // the frame loop
  auto load = [&](int t) -> uint32_t {
    const bool real = t < ps.T;  // uniform
    return load_raw_at<T>(xr, real ? loff : kOutOfRange, real ? t * ps.fstride : 0);
  };
  auto value = [&](int t, uint32_t raw) {
    return (t < ps.T && soff >= 0) ? raw_to_f32<T>(raw) : neutral;
  };
  // frame t's window element sits in xq[t % PF]; the next PF - 1 frames'
  // are in flight while frame t is reduced (one register per frame, so the
  // loop keeps many: it is bound by the latency of these loads)
  constexpr int PF = 16;
  uint32_t xq[PF];
#pragma unroll
  for (int u = 0; u < PF; ++u) {
    xq[u] = load(u);
    __builtin_amdgcn_sched_barrier(0);  // in frame order
  }
  // whole groups of PF frames with no exit inside: frames past the call
  // (the last group's tail) store nothing and leave the window as it is.
  // With a temporal stride the window is still the last kT frames; only
  // every sT-th step from the first emitting one emits (ep: its phase, ko:
  // the outputs so far).
  int ep = 0, ko = 0;
  for (int t0 = 0; t0 < ps.count; t0 += PF) {
#pragma unroll
    for (int u = 0; u < PF; ++u) {
      const int t = t0 + u;
      const bool dead = t >= ps.count;  // uniform
      const float xv = value(t, xq[u]);
      const float val = is_max ? group_max<G>(xv) : group_sum<G>(xv);
      xq[u] = load(t + PF);
      fv[KT - 1] = val;
      fok[KT - 1] = t < ps.T ? 1.f : 0.f;
      const int64_t n = ps.n0 + t;
      {
        // the window's frames as the per-step kernel combines them (tap q in
        // lane q of a lane group, then an xor-shuffle tree), so both paths
        // give the same bits; start padding contributes nothing
        float tv[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) {
          const bool in = q < KT && n - (KT - 1) + q >= 0;
          tv[q] = in ? fv[q < KT ? q : 0] : neutral;
        }
#pragma unroll
        for (int m = 4; m > 0; m >>= 1) {
          float nv[8];
#pragma unroll
          for (int l = 0; l < 8; ++l) nv[l] = is_max ? fmaxf(tv[l], tv[l ^ m]) : tv[l] + tv[l ^ m];
#pragma unroll
          for (int l = 0; l < 8; ++l) tv[l] = nv[l];
        }
        const float acc = tv[0];
        // the count of real frames, only for an average without the pads
        // (uniform branch, no memory operation inside)
        float tcount = 0.f;
        if (!is_max && !g.count_include_pad) {
          float tc[8];
#pragma unroll
          for (int q = 0; q < 8; ++q) {
            const bool in = q < KT && n - (KT - 1) + q >= 0;
            tc[q] = in ? fok[q < KT ? q : 0] : 0.f;
          }
#pragma unroll
          for (int m = 4; m > 0; m >>= 1) {
            float nc[8];
#pragma unroll
            for (int l = 0; l < 8; ++l) nc[l] = tc[l] + tc[l ^ m];
#pragma unroll
            for (int l = 0; l < 8; ++l) tc[l] = nc[l];
          }
          tcount = tc[0];
        }
        float out;
        if (is_max) {
          out = acc;
        } else {
          const float div = g.count_include_pad ? float(KT * kHW) : tcount * float(vh * vw);
          out = div > 0.f ? acc / div : 0.f;
        }
        const bool on = (t >= ps.t_e0) & !dead;  // uniform
        const bool emits = on & (ep == 0);
        store_at(yr, (emits && r == 0) ? yoff : kOutOfRange,
                 emits ? int(int64_t(ko) * So * int64_t(sizeof(T))) : 0, from_f32<T>(out));
        ko += emits ? 1 : 0;
        ep = on ? (ep + 1 == ps.sT ? 0 : ep + 1) : ep;
      }
      // (a dead frame's value went into the last place only, which the next
      // frame overwrites; the call ends after the group anyway)
#pragma unroll
      for (int q = 0; q + 1 < KT; ++q) {
        fv[q] = dead ? fv[q] : fv[q + 1];
        fok[q] = dead ? fok[q] : fok[q + 1];
      }
      __builtin_amdgcn_sched_barrier(0);  // frames in order
    }
  }
  if (ps.update && r == 0) {
    const int64_t n1 = ps.n0 + ps.count;
#pragma unroll
    for (int q = 0; q + 1 < KT; ++q) {
      const int64_t rf = n1 - (KT - 1) + q;
      if (rf >= 0) fifo[(rf % KT) * fifo_slot + idx] = fv[q];
    }
  }
}

// Global spatial pooling (the window covers the whole frame: kH = H, kW = W,
// no spatial padding or dilation, one output per plane and frame), as in a
// network head, over a buffer of frames or a whole clip.  Lanes hold frames
// instead of window positions: a wave stages a block of kPgFrames of a
// plane's frames -- they lie contiguously in the clip -- into LDS with
// 16-byte loads (the next block's, or next plane's, in flight while a block is
// reduced), and lane t reduces frame t of the block alone, in the order of the
// per-step kernel's shuffle tree over 64 window lanes (element r in leaf r,
// the rest neutral), so both paths give the same bits.  The reduced frames
// stay in LDS, the window's span before them first (from the FIFO, then from
// the block before); lane t's window is kT of them, dT apart, combined in the
// per-step kernel's temporal tree (KTB leaves; leaves past kT are neutral, so
// any KTB >= kT gives the same bits).
//
// The call is bound by reading the clip.  A workgroup owns kPgWaves * ppw
// consecutive planes: the FIFO is (slot, plane), so a workgroup reads and
// writes it in runs of up to 16 planes (64 bytes) instead of one float per
// slot.  16 streams x 432 channels, 7x7, 64 frames: a 64-frame average in
// float32 takes 24 us a call (92 MB read and written, 3.8 TB/s; stepping
// through 64 launches took 399 us), and as the second half of a bfloat16
// depthwise + pool clip the whole clip takes 55 us (732 us when each output
// reduced its own 4 x 49 window).
//
// SMALL: planes of at most 16 pixels, in the step kernel's trees of 4 or 16
// leaves (the others are neutral) and with as few staging loads.  SPLIT: the
// calls whose work the form above leaves on too few lanes or CUs.  Calls of at
// most 32 frames take several planes in a pass (lane (pl, tl) is frame tl of
// plane pl): of many planes a block of 64 lanes for each plane costs what 64
// frames cost (65536 planes, two frames, kT 4: 1x1 float32 55 us in one form for
// all, 14 on lane groups, 9.7 here; 8x8 bf16 72, 47 and 9.6).  Clips of few planes
// are cut along time, each piece beginning with the blocks that its windows
// reach back to: one workgroup walks 64 frames in 1.3 to 2 us (one plane, 7x7,
// 20000 frames, kT 4: 613 us in one piece, 35 with a thread per output, 10.6 here).
constexpr int kPgFrames = 64;  // frames per block, one per lane
constexpr int kPgWaves = 4;
constexpr int kPgMaxSpan = 128;  // window span f the LDS history is sized for

struct PoolGlobalArgs {
  int32_t T, count;   // real frames, all frames (the rest end padding)
  int32_t nblk;       // blocks of a plane: ceil(count / kPgFrames)
  int32_t ppw;        // planes per wave
  int32_t planes;     // B * C
  int32_t stage;      // LDS bytes of a wave's staged block
  int32_t F;          // window span f = (kT - 1) dT + 1: FIFO slots
  int32_t hist0;      // first history entry that exists (max(0, F - 1 - n0))
  int32_t slot0;      // n0 mod F
  int32_t t_e0;       // first emitting frame of the call (count: none)
  int32_t update;     // write the FIFO (0: also in clip mode, which has none)
  int32_t x_bytes, y_bytes, fstride;
  FastDiv fd_F, fd_sT;
};

// Split calls.  (A struct of its own: with more arguments, the other form is
// given other registers and measured up to 5% slower.)
struct PoolSplitArgs : PoolGlobalArgs {
  int32_t seg;        // blocks per workgroup (clips: segments of the time axis)
  int32_t warm;       // blocks whose frames reach into the next block's windows
  int32_t pp;         // planes in one pass (short calls)
  int32_t tshift;     // log2 of a plane's lanes: pp << tshift = 64
  int32_t hlen;       // history entries of a plane
};

template <typename T, int KTB, bool IS_MAX, bool SMALL, bool SPLIT>
__global__ __launch_bounds__(64 * kPgWaves) void pool_steps_global_kernel(
    PoolGeom g, typename std::conditional<SPLIT, PoolSplitArgs, PoolGlobalArgs>::type pa,
    const T* __restrict__ x, int64_t x_bc, T* __restrict__ y, int64_t y_bc,
    float* __restrict__ fifo, int64_t fifo_slot, float* __restrict__ valid) {
  extern __shared__ uint4 pg_lds[];
  constexpr uint32_t esz = sizeof(T);
  // 16-byte units per lane and block
  constexpr int NU = (SMALL ? 16 : 64) * int(esz) / 16 + 1;
  constexpr bool is_max = IS_MAX;
  const float neutral = is_max ? -INFINITY : 0.f;
  const int tid = int(threadIdx.x);
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int S = g.H * g.W, F = pa.F, kT = g.kT, dT = g.dT;
  const int per = kPgWaves * pa.ppw;          // planes of this workgroup
  const int bc0 = int(blockIdx.x) * per;
  // only an average over the real frames reads the validity flags
  const bool counted = !is_max && !g.count_include_pad;
  char* lds = reinterpret_cast<char*>(pg_lds);
  char* stage = lds + wave * pa.stage;
  int pp = 1, pl = 0, tl = lane, hlen = F - 1 + kPgFrames;
  int b_out = 0, b_lo = 0, b_hi = pa.nblk;
  if constexpr (SPLIT) {
    // this lane's plane of a pass and frame of a block
    pp = pa.pp;
    pl = lane >> pa.tshift;
    tl = lane & ((1 << pa.tshift) - 1);
    hlen = pa.hlen;
    // this workgroup's blocks: a later segment of a clip first runs through the
    // blocks that its windows reach back to, without emitting
    b_out = int(blockIdx.y) * pa.seg;
    b_lo = max(0, b_out - pa.warm);
    b_hi = min(pa.nblk, b_out + pa.seg);
  }
  float* hist = reinterpret_cast<float*>(lds + kPgWaves * pa.stage);
  float* okay = hist + per * hlen;  // the history's flags, alike for all planes
  const __amdgpu_buffer_rsrc_t xr = make_rsrc(x, pa.x_bytes);
  const __amdgpu_buffer_rsrc_t yr = make_rsrc(y, pa.y_bytes);

  // history entry i of a plane is frame n0 - (F - 1) + i, in slot
  // (n0 + 1 + i) mod F; entries before the stream began are start padding
  for (int e = tid; e < (F - 1) * per; e += 64 * kPgWaves) {
    const int i = e / per, q = e - i * per;
    const int v = pa.slot0 + 1 + i;
    const int slot = v - fdiv(v, pa.fd_F) * F;
    const bool have = i >= pa.hist0 && bc0 + q < pa.planes;
    hist[q * hlen + i] = have ? fifo[int64_t(slot) * fifo_slot + bc0 + q] : neutral;
  }
  if (counted)
    for (int i = tid; i < F - 1; i += 64 * kPgWaves) {
      const int v = pa.slot0 + 1 + i;
      okay[i] = i >= pa.hist0 ? valid[v - fdiv(v, pa.fd_F) * F] : 0.f;
    }
  __syncthreads();

  const int q0 = wave * pa.ppw;
  const int nq = min(pa.ppw, pa.planes - bc0 - q0);  // this wave's planes (<= 0: none)
  auto planes_of = [&](int q) { return min(pp, q0 + nq - q); };

  // block b of local plane q, or all the frames of the pp planes from q on
  // (they lie side by side): its real frames in 16-byte units from the
  // 16-byte boundary at or below their first byte; units past them read the
  // out-of-range offset.  A last unit that would run past the clip's end is
  // left to `tail` single elements, read when the block is staged (once a call)
  struct Block {
    int s0, a0, units, tail;
  };
  auto block = [&](int q, int b) {
    Block k;
    const int t0 = b * kPgFrames;
    const int nr =
        pp > 1 ? planes_of(q) * pa.T : min(max(pa.T - t0, 0), kPgFrames);
    k.s0 = int(uint32_t(bc0 + q) * uint32_t(x_bc) * esz) + t0 * pa.fstride;
    k.a0 = k.s0 & ~15;
    const int bytes = nr > 0 ? k.s0 + nr * pa.fstride - k.a0 : 0;
    const bool whole = k.a0 + ((bytes + 15) & ~15) <= pa.x_bytes;
    k.units = whole ? (bytes + 15) >> 4 : bytes >> 4;
    k.tail = whole ? 0 : (bytes & 15) / int(esz);
    return k;
  };
  auto fetch = [&](const Block& k, uint4 (&v)[NU]) {
#pragma unroll
    for (int j = 0; j < NU; ++j) {
      const int u = j * 64 + lane;
      const auto v4 = __builtin_amdgcn_raw_buffer_load_b128(
          xr, u < k.units ? k.a0 + u * 16 : kOutOfRange, 0, 0);
      v[j] = make_uint4(v4[0], v4[1], v4[2], v4[3]);
    }
  };
  // a wave's LDS operations complete in order: only the compiler has to keep
  // the staged block's writes, its reads and the next block's writes apart
  auto order = [] {
    __builtin_amdgcn_wave_barrier();
    __asm__ volatile("" ::: "memory");
  };
  auto comb = [&](float a, float c) { return is_max ? fmaxf(a, c) : a + c; };

  uint4 v[NU];
  Block cb = block(q0, b_lo);
  if (nq <= 0) cb.units = cb.tail = 0;
  fetch(cb, v);
  for (int q = q0; q < q0 + nq; q += pp) {
    const bool mine = !SPLIT || pl < planes_of(q);
    float* hq = hist + (mine ? q + pl : q) * hlen;
    const int yplane = int(uint32_t(bc0 + q + pl) * uint32_t(y_bc) * esz);
    for (int b = b_lo; b < b_hi; ++b) {
#pragma unroll
      for (int j = 0; j < NU; ++j)
        if (j * 64 + lane < cb.units) reinterpret_cast<uint4*>(stage)[j * 64 + lane] = v[j];
      if (lane < cb.tail) {
        const int off = cb.units * 16 + lane * int(esz);
        if constexpr (esz == 2)
          *reinterpret_cast<uint16_t*>(stage + off) =
              uint16_t(__builtin_amdgcn_raw_buffer_load_b16(xr, cb.a0 + off, 0, 0));
        else
          *reinterpret_cast<uint32_t*>(stage + off) =
              __builtin_amdgcn_raw_buffer_load_b32(xr, cb.a0 + off, 0, 0);
      }
      order();
      const int shift = cb.s0 - cb.a0;
      const bool more = b + 1 < b_hi;
      if (more || q + pp < q0 + nq) {
        cb = more ? block(q, b + 1) : block(q + pp, b_lo);
        fetch(cb, v);
      }

      // lane (pl, tl): frame t0 + tl, its S elements in leaves 0..S-1.  The leaf
      // masks are built from a vector copy of S made here, in the loop: as
      // loop invariants the compiler would hoist all 64 of them, as scalar
      // lane masks, out of the loop and spill them
      int Sv;
      __asm__ volatile("v_mov_b32 %0, %1" : "=v"(Sv) : "s"(S));
      const uint32_t nb = __float_as_uint(neutral);
      const int t = b * kPgFrames + tl;
      const bool real = (t < pa.T) & mine;
      const char* fb = stage + shift + (real ? pl * pa.T + tl : 0) * pa.fstride;
      auto leaf = [&](int r) {
        float xv;
        if constexpr (esz == 2)
          xv = __uint_as_float(uint32_t(*reinterpret_cast<const uint16_t*>(fb + 2 * r)) << 16);
        else
          xv = *reinterpret_cast<const float*>(fb + 4 * r);
        // as the per-step kernel: the neutral value, combined with the element
        const float lv = is_max ? fmaxf(neutral, xv) : neutral + xv;
        const uint32_t keep = uint32_t((r - Sv) >> 31);  // all ones when r < S
        return __uint_as_float((__float_as_uint(lv) & keep) | (nb & ~keep));
      };
      // the tree of the step kernel's lane group; leaves past the smallest
      // group that holds S are neutral and left out
      float red;
      auto tree = [&](auto& tr) __attribute__((always_inline)) {
        constexpr int n = int(sizeof(tr) / sizeof(float));
#pragma unroll
        for (int m = n / 2; m > 0; m >>= 1)
#pragma unroll
          for (int l = 0; l < m; ++l) tr[l] = comb(tr[l], tr[l + m]);
        red = tr[0];
      };
      if constexpr (!SMALL) {
        float tr[32];
        if (S > 32) {  // uniform
#pragma unroll
          for (int l = 0; l < 32; ++l) tr[l] = comb(leaf(l), leaf(l + 32));
        } else {
#pragma unroll
          for (int l = 0; l < 32; ++l) tr[l] = leaf(l);
        }
        tree(tr);
      } else if (S > 4) {  // uniform
        float tr[16];
#pragma unroll
        for (int l = 0; l < 16; ++l) tr[l] = leaf(l);
        tree(tr);
      } else {
        float tr[4];
#pragma unroll
        for (int l = 0; l < 4; ++l) tr[l] = leaf(l);
        tree(tr);
      }
      if (mine) hq[F - 1 + tl] = real ? red : neutral;
      order();

      // the window of frame t: history entries t0 + t + q dT of the block
      // (from a copy of kT made here, for the reason given at the leaves)
      int kTs = kT;
      __asm__ volatile("" : "+s"(kTs));
      float tv[KTB];
#pragma unroll
      for (int a = 0; a < KTB; ++a) {
        tv[a] = neutral;
        if (a < kTs) tv[a] = hq[tl + a * dT];  // uniform
      }
#pragma unroll
      for (int m = KTB / 2; m > 0; m >>= 1)
#pragma unroll
        for (int l = 0; l < m; ++l) tv[l] = comb(tv[l], tv[l + m]);
      float out = tv[0];
      if constexpr (!is_max) {
        float div = float(kT * S);
        if (counted) {
          float cnt = 0.f;  // whole numbers: any order
          for (int a = 0; a < kT; ++a) {
            const int e = b * kPgFrames + tl + a * dT - (F - 1);  // frame of the call
            cnt += e < 0 ? okay[F - 1 + e] : e < pa.T ? 1.f : 0.f;
          }
          div = cnt * float(S);
        }
        out = div > 0.f ? out / div : 0.f;
      }
      const int te = t - pa.t_e0;
      const int k = te >= 0 ? fdiv(te, pa.fd_sT) : 0;  // the call's k-th output
      const bool emits =
          mine && (!SPLIT || b >= b_out) && t < pa.count && te >= 0 && te == k * g.sT;
      store_at(yr, emits ? yplane + k * int(esz) : kOutOfRange, 0, from_f32<T>(out));

      // the span before the next block: the block's last F - 1 frames (a pass
      // over several planes is the call's only one: its span stays in place)
      if (pp > 1) break;
      const int nf = min(kPgFrames, pa.count - b * kPgFrames);
      for (int i0 = 0; i0 < F - 1; i0 += 64) {
        const int i = i0 + lane;
        const float h = hq[min(i, F - 2) + nf];
        order();
        if (i < F - 1) hq[i] = h;
        order();
      }
    }
  }
  if (!pa.update) return;
  __syncthreads();
  // the call's last F - 1 frames go to their FIFO slots: history entry i is
  // frame n0 + count - (F - 1) + i
  const int first = max(0, F - 1 - pa.count);
  const int at = pp > 1 ? pa.count : 0;
  for (int e = first * per + tid; e < (F - 1) * per; e += 64 * kPgWaves) {
    const int i = e / per, q = e - i * per;
    const int v = pa.slot0 + pa.count + 1 + i;
    const int slot = v - fdiv(v, pa.fd_F) * F;
    if (bc0 + q < pa.planes) fifo[int64_t(slot) * fifo_slot + bc0 + q] = hist[q * hlen + at + i];
  }
  // nobody reads the flags of this layer in this launch (otherwise they are
  // written by a launch of their own)
  if (!counted && blockIdx.x == 0)
    for (int t = max(0, pa.count - F) + tid; t < pa.count; t += 64 * kPgWaves) {
      const int v = pa.slot0 + t;
      valid[v - fdiv(v, pa.fd_F) * F] = t < pa.T ? 1.f : 0.f;
    }
}

// Validity flags of the FIFO slots the call's frames went to (one wave; the
// last R frames have a slot each).
__global__ void pool_valid_kernel(float* valid, int32_t R, int64_t n0, int32_t count, int32_t T) {
  const int32_t first = count > R ? count - R : 0;
  for (int32_t t = first + int32_t(threadIdx.x); t < count; t += 64)
    valid[(n0 + t) % R] = t < T ? 1.f : 0.f;
}

__global__ void pool_header_kernel(StateHeader h, StateHeader* dst) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *dst = h;
}

template <typename T, int G>
hipError_t pool_step_g(const PoolGeom& g, const PoolLayout& L, char* state, const StepIO& io,
                       const co_pool_plan& plan, bool update, bool pad, hipStream_t s) {
  PoolTaps taps;
  for (int j = 0; j < CO_MAX_TAPS; ++j) taps.src[j] = plan.src[j];
  float* fifo = reinterpret_cast<float*>(state + L.fifo);
  float* valid = reinterpret_cast<float*>(state + L.valid);
  hipLaunchKernelGGL((pool_step_kernel<T, G>), dim3(grid_for(g.out_frame_elems() * G)),
                     dim3(kBlock), 0, s, g, static_cast<const T*>(io.x), io.x_bc,
                     static_cast<T*>(io.y), io.y_bc, fifo, L.fifo_slot_elems, valid,
                     plan.write_slot, update ? 1 : 0, plan.emit, pad ? 1 : 0, taps,
                     make_fastdiv(uint32_t(g.So())), make_fastdiv(uint32_t(g.Wo)),
                     make_fastdiv(uint32_t(g.kW)));
  return hipGetLastError();
}

// Lanes per output element: enough to cover the spatial window (and the
// temporal taps) in about one load each.
template <typename T>
hipError_t pool_step_t(const PoolGeom& g, const PoolLayout& L, char* state, const StepIO& io,
                       const co_pool_plan& plan, bool update, bool pad, hipStream_t s) {
  const int work = std::max(g.kH * g.kW, g.kT);
  if (work > 16) return pool_step_g<T, 64>(g, L, state, io, plan, update, pad, s);
  if (work > 4) return pool_step_g<T, 16>(g, L, state, io, plan, update, pad, s);
  return pool_step_g<T, 4>(g, L, state, io, plan, update, pad, s);
}

}  // namespace

hipError_t launch_pool_step(const PoolGeom& g, const PoolLayout& L, char* state,
                            const StepIO& io, const co_pool_plan& plan, bool update_state,
                            bool pad_frame, hipStream_t s) {
  if (g.dtype == CO_BF16) return pool_step_t<bf16_t>(g, L, state, io, plan, update_state, pad_frame, s);
  return pool_step_t<float>(g, L, state, io, plan, update_state, pad_frame, s);
}

hipError_t launch_pool_init(const PoolGeom& g, const PoolLayout& L, char* state,
                            const StateHeader& hdr, hipStream_t s) {
  hipLaunchKernelGGL(pool_header_kernel, dim3(1), dim3(64), 0, s, hdr,
                     reinterpret_cast<StateHeader*>(state + L.header));
  return hipGetLastError();
}

namespace {

// Global spatial pooling over small frames (H * W <= 64: one window element
// per lane of the per-step kernel's groups) with a window span the kernel's
// history holds: the frames-in-lanes kernel, any temporal stride and dilation.
bool pool_global_fits(const PoolGeom& g) {
  return g.kH == g.H && g.kW == g.W && g.pH == 0 && g.pW == 0 && g.dH == 1 && g.dW == 1 &&
         g.H * g.W <= 64 && g.kT <= 64 && g.f <= kPgMaxSpan;
}

template <typename T, bool IS_MAX, bool SMALL>
auto pool_global_pick(int kT) {
  return kT <= 8    ? pool_steps_global_kernel<T, 8, IS_MAX, SMALL, false>
         : kT <= 16 ? pool_steps_global_kernel<T, 16, IS_MAX, SMALL, false>
         : kT <= 32 ? pool_steps_global_kernel<T, 32, IS_MAX, SMALL, false>
                    : pool_steps_global_kernel<T, 64, IS_MAX, SMALL, false>;
}

// Split calls come with the smallest and the largest temporal tree only.
template <typename T, bool IS_MAX, bool SMALL>
auto pool_split_pick(int kT) {
  return kT <= 8 ? pool_steps_global_kernel<T, 8, IS_MAX, SMALL, true>
                 : pool_steps_global_kernel<T, 64, IS_MAX, SMALL, true>;
}

// state null: clip mode (a stream that begins and ends with the clip).
template <typename T>
hipError_t pool_global_t(const PoolGeom& g, const PoolLayout& L, char* state, const void* x,
                         int64_t x_bc, int32_t nreal, int32_t count, void* y, int64_t y_bc,
                         int64_t n0, bool update, hipStream_t s) {
  const int64_t esz = g.dtype == CO_BF16 ? 2 : 4;
  PoolSplitArgs pa;
  pa.T = nreal;
  pa.count = count;
  pa.nblk = int32_t((int64_t(count) + kPgFrames - 1) / kPgFrames);
  pa.planes = int32_t(int64_t(g.B) * g.C);
  pa.F = g.f;
  // short calls: as many planes in a pass as have frames for the lanes (they
  // are staged in one run)
  pa.tshift = 6;
  pa.pp = 1;
  while (pa.tshift > 0 && 1 << (pa.tshift - 1) >= count && x_bc == nreal * g.S()) {
    --pa.tshift;
    pa.pp *= 2;
  }
  // planes per wave: runs of 16 planes of the FIFO per workgroup where that
  // leaves a workgroup per CU, else more workgroups
  pa.ppw = std::max(4, pa.pp);
  while (pa.ppw > 1 && pa.planes / (kPgWaves * pa.ppw) < 256) pa.ppw /= 2;
  if (pa.pp > pa.ppw) {
    pa.pp = pa.ppw;
    pa.tshift = 6 - __builtin_ctz(unsigned(pa.pp));
  }
  pa.hlen = pa.F - 1 + (1 << pa.tshift);
  pa.hist0 = int32_t(std::max<int64_t>(0, g.f - 1 - n0));
  pa.slot0 = int32_t(n0 % g.f);
  const int64_t te = n0 >= g.d ? (g.sT - (n0 - g.d) % g.sT) % g.sT : g.d - n0;
  pa.t_e0 = int32_t(std::min<int64_t>(te, count));
  pa.update = update && state ? 1 : 0;
  pa.x_bytes = int32_t(((int64_t(g.B) * g.C - 1) * x_bc + int64_t(nreal) * g.S()) * esz);
  pa.y_bytes = int32_t(int64_t(g.B) * g.C * y_bc * esz);
  pa.fstride = int32_t(g.S() * esz);
  pa.fd_F = make_fastdiv(uint32_t(g.f));
  pa.fd_sT = make_fastdiv(uint32_t(g.sT));
  // a block, its alignment shift and the 64-element over-read of the last lane
  const int64_t rows = std::min<int64_t>(kPgFrames, int64_t(nreal) * pa.pp);
  pa.stage = int32_t(((rows * g.S() + 64) * esz + 32 + 15) / 16 * 16);
  const int per = kPgWaves * pa.ppw;
  const int lds = kPgWaves * pa.stage + (per * pa.hlen + pa.F) * 4;
  // a clip has no FIFO: where its planes leave CUs without work, its blocks go
  // to several workgroups, each at least twice as long as its warm-up
  const int64_t wgs = (int64_t(pa.planes) + per - 1) / per;
  pa.warm = (pa.F - 1 + kPgFrames - 1) / kPgFrames;
  int64_t segs = 1;
  if (!state)
    segs = std::max<int64_t>(1, std::min<int64_t>(1024 / wgs, pa.nblk / std::max(1, 2 * pa.warm)));
  pa.seg = int32_t((pa.nblk + segs - 1) / segs);
  segs = (pa.nblk + pa.seg - 1) / std::max(pa.seg, 1);
  float* fifo = state ? reinterpret_cast<float*>(state + L.fifo) : nullptr;
  float* valid = state ? reinterpret_cast<float*>(state + L.valid) : nullptr;
  const bool small = g.S() <= 16, max = g.kind == CO_POOL_MAX;
  auto launch = [&](auto kern, const auto& args) {
    if (lds > 64 * 1024) {
      const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                               hipFuncAttributeMaxDynamicSharedMemorySize, lds);
      if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(kern, dim3(unsigned(wgs), unsigned(std::max<int64_t>(segs, 1))),
                       dim3(64 * kPgWaves), lds, s, g, args, static_cast<const T*>(x), x_bc,
                       static_cast<T*>(y), y_bc, fifo, L.fifo_slot_elems, valid);
    return hipGetLastError();
  };
  hipError_t e;
  if (pa.pp > 1 || segs > 1)
    e = launch(max && small ? pool_split_pick<T, true, true>(g.kT)
               : max        ? pool_split_pick<T, true, false>(g.kT)
               : small      ? pool_split_pick<T, false, true>(g.kT)
                            : pool_split_pick<T, false, false>(g.kT),
               pa);
  else
    e = launch(max && small ? pool_global_pick<T, true, true>(g.kT)
               : max        ? pool_global_pick<T, true, false>(g.kT)
               : small      ? pool_global_pick<T, false, true>(g.kT)
                            : pool_global_pick<T, false, false>(g.kT),
               static_cast<const PoolGlobalArgs&>(pa));
  if (e != hipSuccess || !pa.update) return e;
  if (g.kind == CO_POOL_MAX || g.count_include_pad) return e;  // written in the launch
  hipLaunchKernelGGL(pool_valid_kernel, dim3(1), dim3(64), 0, s, valid, g.R, n0, count, nreal);
  return hipGetLastError();
}

template <typename T, int G, int KT>
hipError_t pool_steps_launch(const PoolGeom& g, const PoolLayout& L, char* state, const void* x,
                             int64_t x_bc, int32_t nreal, int32_t count, void* y, int64_t y_bc,
                             int64_t n0, bool update, hipStream_t s) {
  PoolSteps ps;
  ps.n0 = n0;
  ps.count = count;
  ps.T = nreal;
  ps.emit0 = n0 > g.d ? n0 : g.d;
  ps.sT = g.sT;
  {
    const int64_t te = n0 >= g.d ? (g.sT - (n0 - g.d) % g.sT) % g.sT : g.d - n0;
    ps.t_e0 = int32_t(std::min<int64_t>(te, count));
  }
  ps.update = update ? 1 : 0;
  const int64_t esz = g.dtype == CO_BF16 ? 2 : 4;
  ps.x_bytes = int32_t(((int64_t(g.B) * g.C - 1) * x_bc + int64_t(nreal) * g.S()) * esz);
  ps.y_bytes = int32_t(int64_t(g.B) * g.C * y_bc * esz);
  ps.fstride = int32_t(g.S() * esz);
  ps.fd_So = make_fastdiv(uint32_t(g.So()));
  ps.fd_Wo = make_fastdiv(uint32_t(g.Wo));
  ps.fd_kW = make_fastdiv(uint32_t(g.kW));
  float* fifo = reinterpret_cast<float*>(state + L.fifo);
  float* valid = reinterpret_cast<float*>(state + L.valid);
  auto kern = g.kind == CO_POOL_MAX ? pool_steps_kernel<T, G, KT, true>
                                     : pool_steps_kernel<T, G, KT, false>;
  hipLaunchKernelGGL(kern, dim3(grid_for(g.out_frame_elems() * G)), dim3(kBlock), 0, s, g, ps,
                     static_cast<const T*>(x), x_bc, static_cast<T*>(y), y_bc, fifo,
                     L.fifo_slot_elems, valid);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || !update) return e;
  hipLaunchKernelGGL(pool_valid_kernel, dim3(1), dim3(64), 0, s, valid, g.R, n0, count, nreal);
  return hipGetLastError();
}

template <typename T, int G>
hipError_t pool_steps_kt(const PoolGeom& g, const PoolLayout& L, char* state, const void* x,
                         int64_t x_bc, int32_t nreal, int32_t count, void* y, int64_t y_bc,
                         int64_t n0, bool update, hipStream_t s) {
  switch (g.kT) {
    case 1: return pool_steps_launch<T, G, 1>(g, L, state, x, x_bc, nreal, count, y, y_bc, n0, update, s);
    case 2: return pool_steps_launch<T, G, 2>(g, L, state, x, x_bc, nreal, count, y, y_bc, n0, update, s);
    case 3: return pool_steps_launch<T, G, 3>(g, L, state, x, x_bc, nreal, count, y, y_bc, n0, update, s);
    case 4: return pool_steps_launch<T, G, 4>(g, L, state, x, x_bc, nreal, count, y, y_bc, n0, update, s);
    case 5: return pool_steps_launch<T, G, 5>(g, L, state, x, x_bc, nreal, count, y, y_bc, n0, update, s);
    default: return hipErrorInvalidValue;
  }
}

template <typename T>
hipError_t pool_steps_t(const PoolGeom& g, const PoolLayout& L, char* state, const void* x,
                        int64_t x_bc, int32_t nreal, int32_t count, void* y, int64_t y_bc,
                        int64_t n0, bool update, hipStream_t s) {
  if (pool_global_fits(g))
    return pool_global_t<T>(g, L, state, x, x_bc, nreal, count, y, y_bc, n0, update, s);
  const int kHW = g.kH * g.kW;
  if (kHW > 16) return pool_steps_kt<T, 64>(g, L, state, x, x_bc, nreal, count, y, y_bc, n0, update, s);
  if (kHW > 4) return pool_steps_kt<T, 16>(g, L, state, x, x_bc, nreal, count, y, y_bc, n0, update, s);
  return pool_steps_kt<T, 4>(g, L, state, x, x_bc, nreal, count, y, y_bc, n0, update, s);
}

}  // namespace

hipError_t launch_pool_valid(float* valid, int32_t R, int64_t n0, int32_t count, int32_t T,
                             hipStream_t s) {
  hipLaunchKernelGGL(pool_valid_kernel, dim3(1), dim3(64), 0, s, valid, R, n0, count, T);
  return hipGetLastError();
}

bool pool_steps_supported(const PoolGeom& g, int64_t x_frames, int64_t y_frames) {
  const int64_t esz = g.dtype == CO_BF16 ? 2 : 4;
  // the lane-group kernel's window is the last kT <= 5 frames: any temporal
  // stride, no dilation
  const bool group = g.dT == 1 && g.kT >= 1 && g.kT <= 5 && g.kH * g.kW <= 64;
  return (pool_global_fits(g) || group) &&
         int64_t(g.B) * g.C * x_frames * g.S() * esz < (int64_t(1) << 31) &&
         int64_t(g.B) * g.C * y_frames * g.So() * esz < (int64_t(1) << 31);
}

hipError_t launch_pool_steps(const PoolGeom& g, const PoolLayout& L, char* state, const void* x,
                             int64_t x_bc, int32_t nreal, int32_t count, void* y, int64_t y_bc,
                             int64_t n0, bool update, hipStream_t s) {
  if (g.dtype == CO_BF16)
    return pool_steps_t<bf16_t>(g, L, state, x, x_bc, nreal, count, y, y_bc, n0, update, s);
  return pool_steps_t<float>(g, L, state, x, x_bc, nreal, count, y, y_bc, n0, update, s);
}

hipError_t launch_pool_clip(const PoolGeom& g, int32_t T, int32_t T_out, const void* x, void* y,
                            hipStream_t s) {
  const int64_t total = int64_t(g.B) * g.C * T_out * g.So();
  if (total == 0) return hipSuccess;
  // a clip is a stream that begins with it and ends with its end padding
  // (Principles 2 and 4), so the frames-in-lanes kernel serves it without a
  // state; other windows reduce every output's window on its own
  // A window over single pixels is kT values, and threads beside each other read
  // values beside each other: for a few of them and a million outputs a thread
  // per output is the faster (16 x 432 planes, float32: 2000 frames, kT 1 51 us
  // against 70, kT 4 84 against 78; 300 frames, kT 4 14.6 against 16.7, kT 16
  // 31 against 26; 432 planes of 2000 frames 9.6 against 9).
  const bool single =
      g.S() == 1 && g.kT <= (T < 1024 ? 4 : 2) && total >= (int64_t(1) << 20);
  if (!single && pool_global_fits(g) && pool_steps_supported(g, T, T_out)) {
    const auto launch = g.dtype == CO_BF16 ? pool_global_t<bf16_t> : pool_global_t<float>;
    return launch(g, PoolLayout{}, nullptr, x, int64_t(T) * g.S(), T, T + g.pT, y,
                  int64_t(T_out), 0, false, s);
  }
  if (g.dtype == CO_BF16)
    hipLaunchKernelGGL(pool_clip_kernel<bf16_t>, dim3(grid_for(total)), dim3(kBlock), 0, s, g, T,
                       T_out, static_cast<const bf16_t*>(x), static_cast<bf16_t*>(y));
  else
    hipLaunchKernelGGL(pool_clip_kernel<float>, dim3(grid_for(total)), dim3(kBlock), 0, s, g, T,
                       T_out, static_cast<const float*>(x), static_cast<float*>(y));
  return hipGetLastError();
}

}  // namespace coinf
