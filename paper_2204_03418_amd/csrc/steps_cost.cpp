// What a forward_steps call of a matrix-core layer costs by each of the ways
// that it can run: as one GEMM over its frames (conv_clip.hip), as one
// persistent launch (conv_reg.hip, conv_gemm.hip) or as a loop of single steps.
// All of them give the same bits, so the choice is by time alone.
//
// The ways differ by what they pay once.  The GEMM over frames spreads a call
// over the chip whatever its length, but walks K = kT x taps x channels in one
// chain, and once more for the outputs that the call leaves unfinished: 15 to
// 550 us before the first frame counts.  A persistent kernel loads its weights
// once and then walks the frames.  A step is a launch.  Short calls are for the
// loop, long ones for the GEMM, and the persistent kernels are between them.
//
// The terms are those of the kernels' structure, the constants are fitted to
// times measured on MI355X: 1924 calls of 29 layers (skeleton, pointwise and
// video layers, 24 to 432 channels, kT 1 to 9, temporal stride 1 and 2, both
// dtypes) with 1 to 64 streams and 2 to 300 frames, whose frames change from
// call to call.  A clip of 300 frames beyond about 100 MB counts with the mean
// of changing and of repeated frames: the bf16 persistent kernels gain a third
// from frames that the memory-side cache holds, the GEMM a tenth.  Taking the
// cheapest by these estimates costs 0.5% over the best way on average, less than
// 1% in 95 of 100 calls and 1.3x in the worst.
#include <algorithm>

#include "launch.hpp"
#include "schedule.hpp"

namespace coinf {

bool clip_unpadded(const ConvGeom& g) { return g.kH * g.kW == 1 && g.pH == 0 && g.pW == 0; }

bool clip_pairs(const ConvGeom& g) {
  return g.dtype == CO_BF16 && g.kH * g.kW == 1 && g.sT == 1 && g.sH == 1 && g.sW == 1 &&
         g.pH == 0 && g.pW == 0;
}

namespace {

// Workgroups of `tile` channels that `outputs` output frames take.
int64_t clip_wgs(const ConvGeom& g, int64_t outputs, int tile) {
  return ceil_div(outputs * g.So(), 128) * g.B * ceil_div(g.Cout, tile);
}

// Every call: its launch and what the host does around it.
constexpr double kCallUs = 9.7;

}  // namespace

// Channel tile: the least padded width times (1 + what a tile's input staging
// costs against its matrix work, about 32 channels' worth).  Where bf16
// gathers pixel by pixel and there is work for two workgroups a CU, 192
// channels take the taller wave tile (128 x 48): the waves of a workgroup then
// share no weights, and a weight fragment fetched through L1 feeds eight
// instructions instead of four (64 streams, 192 -> 192, 3x3x3, 14x14, 16
// frames: 667 us against 1010 us in 96-channel tiles; 16 streams, 8 frames:
// 229 against 219).
int clip_tile(const ConvGeom& g, int64_t outputs) {
  int best = 0;
  int64_t cost = 0;
  for (const int n : {32, 64, 96, 128}) {
    const int64_t c = ceil_div(g.Cout, n) * (n + 32);
    if (best == 0 || c < cost) {
      best = n;
      cost = c;
    }
  }
  if (best == 96 && g.dtype == CO_BF16 && !clip_pairs(g) && clip_wgs(g, outputs, 192) >= 512 &&
      ceil_div(g.Cout, 192) * 192 <= ceil_div(g.Cout, 96) * 96)
    return 192;
  return best;
}

// The GEMM over frames.  A k-step takes its latency (mostly the wave tile's
// matrix instructions in float32, the operands' way in bf16) while the CUs have
// a workgroup each, and beyond that `rate` for every workgroup on the fullest
// CU, in proportion to its channels (bf16 tiles narrower than 96 channels cost
// as much).  The second pass (tail: the state is updated) walks the taps of the
// unfinished outputs and writes the ring, which calls shorter than kT, all of
// whose outputs began before them, read first.
double clip_us(const ConvGeom& g, int64_t frames, bool tail) {
  struct Fit {
    double start, second, latency, per_tile, rate, open, ring_mb;
  };
  const bool bf = g.dtype == CO_BF16;
  const Fit f = !bf             ? Fit{6.67, 1.66, 0.312, 0.906, 1.015, 0.68, 0.60}
                : clip_pairs(g) ? Fit{7.86, 3.75, 0.131, 0.406, 0.355, 2.68, 0.67}
                                : Fit{6.58, 2.81, 0.439, 0.267, 0.447, 0.14, 0.61};
  const int64_t outputs = ceil_div(frames, g.sT);
  const int tile = clip_tile(g, outputs);
  const double q = double(g.kH) * g.kW * ceil_div(g.Cin, bf ? 32 : 16);
  const double wide = double(bf ? std::max(tile, 96) : tile) / 128;
  const double latency = f.latency + f.per_tile * tile / 128;
  auto ksteps = [&](double taps, int64_t outs) {
    return taps * q *
           std::max(latency, f.rate * wide * double(ceil_div(clip_wgs(g, outs, tile), 256)));
  };
  double us = f.start + ksteps(double(std::min<int64_t>(g.kT, frames)), outputs);
  if (tail && g.kT > 1) {
    const int64_t open = ceil_div(g.kT - 1, g.sT);  // unfinished outputs
    const int64_t taps = std::min<int64_t>(g.kT - 1, frames + (open - 1) * g.sT);
    const double ring = f.ring_mb * 4e-6 * double(g.R) * g.B * g.So() * g.Cout;
    us += f.second + ksteps(double(taps), g.R) + ring;
    if (frames < g.kT) us += f.open + ring;
  }
  return std::max(us, kCallUs);
}

// Single steps: a launch, or what its kernel takes.  The register GEMM's time
// goes with the waves that a SIMD gets and the k-steps of a wave.
double loop_us(const ConvGeom& g, int64_t frames) {
  double us;
  RegConfig r;
  if (g.algo == CO_ALGO_GEMM_REG) {
    if (!reg_config(g, g.cfg, &r)) return 0;
    struct Fit {
      double start, wave, kstep;
    };
    const Fit f = r.id == 0   ? Fit{5.38, 0.415, 0.108}
                  : r.id == 1 ? Fit{4.47, 1.245, 0.023}
                  : r.id == 5 ? Fit{4.47, 0.733, 0.497}
                  : r.id == 6 ? Fit{3.70, 1.025, 0.107}
                  : r.id == 7 ? Fit{4.39, 1.350, 0.172}
                  : r.id == 8 ? Fit{4.78, 2.292, 0.034}
                  : r.id == 9 ? Fit{3.71, 0.533, 0.159}
                              : Fit{4.60, 1.200, 0};
    const double waves = double(r.m_frags) * ceil_div(r.n_frags, r.WN) * r.KSPLIT / g.sT;
    us = f.start + waves / 1024 * (f.wave + f.kstep * r.KS);
  } else {
    GemmConfig c;
    if (!gemm_config(g, g.cfg, &c)) return 0;
    const double taps = double(g.kH) * g.kW, chunks = c.n_chunks;
    if (c.M_WG == 448) {
      const double mflops = 2e-6 * g.B * g.So() * g.Cout * g.kT * g.Cin * taps / g.sT;
      us = 9 + 0.21 * taps * chunks + mflops / 1450;
    } else {
      // tiles of 32 x 128 (bf16, float32) and 64 x 16 (float32): a chunk of
      // channels takes its latency, or the fullest CU its tiles
      struct Fit {
        double l0, l1, tile, r0, r1;
      };
      const Fit f = g.dtype == CO_BF16 ? Fit{0.530, 0.136, 5.44, 0, 0.136}
                    : c.N_WG == 128    ? Fit{0.800, 0.341, 0.95, 0.410, 0.210}
                                       : Fit{0.636, 0.051, 1.37, 0.161, 0.082};
      const double tiles = double(c.m_tiles) * ceil_div(c.n_tiles, g.sT) / 256;
      us = 5 + std::max(chunks * (f.l0 + f.l1 * taps),
                        tiles * (f.tile + chunks * (f.r0 + f.r1 * taps)));
    }
  }
  return std::max(6 + 3.6 * frames, 1 + double(frames) * std::max(us, 5.1));
}

// The register GEMM's persistent kernels of one spatial tap (conv_reg.hip):
// weights into registers, then frame after frame, in the time segments that
// the launch deals to the waves the chip holds, and the call's bytes.
double reg_steps_us(const ConvGeom& g, const RegConfig& c, int64_t frames) {
  const bool bf = g.dtype == CO_BF16, plain = g.sT == 1 && g.dT == 1;
  const double work = double(g.kT) * c.CS;
  const double mb = 1e-6 * (bf ? 2 : 4) * g.B *
                    (double(frames) * g.Cin * g.S() + double(ceil_div(frames, g.sT)) * g.Cout * g.So());
  // waves of a workgroup and of a SIMD, frames before a segment
  const int64_t sw = plain && c.id == 5 ? 8 : 4, wpe = !plain || c.id == 5 ? 2 : 1;
  const int64_t warm = plain ? g.kT - 1 : std::max((g.kT - 1) * g.dT, g.sT * g.R);
  const int64_t wgs = int64_t(c.m_frags) * ceil_div(ceil_div(g.Cout, 16), sw);
  int64_t segs = wpe * 1024 / std::max<int64_t>(wgs * sw, 1);
  if (warm > 0) segs = std::min<int64_t>(segs, frames / (4 * warm));
  segs = std::max<int64_t>(1, std::min<int64_t>(segs, 64));
  const int64_t len = ceil_div(frames, segs);
  segs = ceil_div(frames, std::max<int64_t>(len, 1));
  const double walk = double(len + (segs > 1 ? warm : 0));
  const double waves = double(wgs * sw * segs);
  if (!plain) {
    const double frame = bf ? 0.054 * work : 0.98 + 0.005 * work;
    const double share = 1 + (bf ? 0.146 : 0.863) * std::max(0.0, waves / 1024 - 1);
    return std::max(kCallUs, 7.6 + walk * frame * share + (bf ? 0.159 : 0.0) * mb);
  }
  struct Fit {
    double start, once, load, frame, per, mb;
  };
  const Fit f = c.id == 0   ? Fit{8.00, 0, 0.131, 0.300, 0.011, 0.300}
                : c.id == 1 ? Fit{7.60, 0.039, 0.039, 1.451, 0, 0.196}
                : c.id == 5 ? Fit{8.00, 0.168, 0.168, 0.300, 0, 0.347}
                            : Fit{8.05, 0.131, 0.131, 0.651, 0, 0};
  const double rounds = double(ceil_div(wgs * sw * segs, 1024 * wpe));
  return std::max(kCallUs, f.start + f.once * work +
                               rounds * (f.load * work + walk * (f.frame + f.per * work)) +
                               f.mb * mb);
}

// The persistent 3x3 GEMM: about 3.2 us a frame and 32 channels for every 256
// workgroups (160 pixels x 64 channels).
double gemm_steps_us(const GemmStepsConfig& c, int64_t frames) {
  const double rounds = double(ceil_div(int64_t(c.m_tiles) * c.o_tiles, 256));
  return 8 + double(frames) * rounds * c.n_chunks * 3.2;
}

StepsRoute cheapest_steps(const ConvGeom& g, int64_t frames, StepsMode mode, bool clip, bool gemm,
                          bool reg) {
  // One temporal tap: nothing to keep on chip, and the GEMM over frames is 2.5x
  // to 4.9x as fast as the persistent kernels (for a pointwise layer 10 us
  // against 14 already for two steps).  Their plain form is also left
  // out at a kT between those it is built for (18 joints, 64 -> 256, kT 5, 64
  // streams, 16 frames: 48 us against 29).
  if (clip && frames >= 2 && g.kT == 1 && g.kH * g.kW == 1) return StepsRoute::Clip;
  RegConfig c;
  const bool one_tap = reg && reg_config(g, g.cfg, &c) && c.TAPS == 1;
  if (clip && g.kT == 1) reg = gemm = false;
  if (clip && one_tap && g.sT == 1 && g.dT == 1 && g.kT != 3 && (g.kT != 9 || c.id == 1))
    reg = false;
  // without updating the state, a loop saves the ring before and restores it
  // after (two copies and an allocation)
  StepsRoute best = StepsRoute::Loop;
  double us = loop_us(g, frames) + (mode == StepsMode::Peek ? 32 : 0);
  auto offer = [&](bool can, StepsRoute r, double t) {
    if (can && t < us) {
      best = r;
      us = t;
    }
  };
  if (reg) {
    // 3x3 shapes keep partial sums and weights in registers: 18 us against the
    // GEMM's 27 (24 -> 24, 56x56, 4 streams, 2 frames), 59 against 54 (16)
    if (!one_tap) return StepsRoute::Reg;
    offer(true, StepsRoute::Reg, reg_steps_us(g, c, frames));
  }
  GemmStepsConfig sc;
  offer(gemm && gemm_steps_config(g, &sc), StepsRoute::Gemm, gemm ? gemm_steps_us(sc, frames) : 0);
  offer(clip, StepsRoute::Clip, clip_us(g, frames, mode == StepsMode::Update));
  return best;
}

}  // namespace coinf
