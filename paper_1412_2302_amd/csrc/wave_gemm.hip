// Launchers of the small products (gemm_wave.h): which layers take them, and their grids.
#include <algorithm>
#include <cmath>

#include "fc_epilogue.h"
#include "gemm_wave.h"
#include "kernels.h"

namespace ax {

// Time of a product in ns slices, by steps of 16 k and one tile: a compute unit does one in about a tenth of a microsecond,
// fp32, however many waves share it, and ends with the others.  Measured (steps, workgroups, us): 13, 6728, 39.5; 13, 3136,
// 22.5; 144, 72, 14; 256, 32, 28; the two gradients of 122 K steps in 3640 workgroups 49.6.  bf16: 13, 3364, 16.5; 13, 1568,
// 10.4.  The planners of conv_gemm.hip are as close (39 us for the first of these in 128 x 64 tiles, where they say 41),
// except below ten microseconds, where they are too low.
constexpr double kWaveLaunch = 4e-6, kWaveStep = 0.1e-6, kWaveStep16 = 0.07e-6, kWaveFinish = 4e-6;
static double wave_seconds(double blocks, double steps, bool bf) {
  return kWaveLaunch + (bf ? kWaveStep16 : kWaveStep) * steps * std::ceil(blocks / 256);
}
// bf16 tiles the planner has at 7 us took 13 (36 workgroups), and have weights converted for them first; weight gradients of
// 16 output channels 29 where it has 19.
// For a stage of a bf16 handle this is a line drawn by whole steps.  tile_seconds_...() has forward products and data gradients
// from the kernels over stored operands, but weight gradients and dense layers from those of gemm_bf16.h, which fp32 operands
// would run on; the direct ones take half of that.  By products alone stages would leave much earlier (mini net, second layer,
// 128 pictures, both gradients: 24 us here, 14 there), but the first to leave brings the side stream, its events and three
// conversions with it: a step of 128 pictures takes 176 us with small products only, 289 with the gradients in tiles, 270
// without any; of 200 210, 329, 332.  From 214 pictures on, where this line ends it (midi net: 380), small products only would
// still be faster for a while: 256 282 | 253, 400 338 | 330, 450 361 | 356, 512 383 | 406, midi net 450 270 | 229.
static double tile_floor(double seconds, bool bf, double below = 18e-6, double extra = 5e-6) {
  return bf && seconds < below ? seconds + extra : seconds;
}
constexpr double kWeightBelow = 25e-6;
struct WavePlan {
  int ns;
  double blocks, steps;  // of the launch; of a workgroup
  double seconds;
};
// Waves per workgroup, for a launch of so many workgroups whose longest reduction has so many steps
static int wave_count(double blocks, double steps) {
  if (blocks <= 256 && steps > 8) return 16;
  return blocks <= 512 && steps > 4 ? 8 : 4;
}
// The chain of steps that one wave of so many has, at `link` seconds each; counts where it outlasts the chip's share of the work.
static double chain_seconds(double steps, int waves, double link) { return kWaveLaunch + std::ceil(steps / waves) * link; }
// of a data gradient: a lane reads 32 bytes of a row of og weights at a time, and past a cache line each lane's row is in a line
// of its own (rows of 128 bytes and less, mini and midi net: 0.7 to 0.85 us a step)
static double data_link(const ConvGeom& c) { return c.og() > 32 ? 1.3e-6 : 0.8e-6; }
// max_k: longest slice the tables hold
static WavePlan wave_plan(long M, long N, long K, int groups, bool bf, long max_k, double link = 0) {
  const double blocks = (double)ceil_div(M, kWaveTile) * ceil_div(N, kWaveTile) * groups;
  const int steps = ceil_div(K, 16), least = ceil_div(K, max_k);
  WavePlan best{least, 0, 0, 1e30};
  for (int ns = least; ns <= least + 15; ++ns) {
    const int per = ceil_div(steps, ns);
    if (ns > least && (per < 4 || ceil_div(steps, per) != ns)) continue;
    const double t = std::max(wave_seconds(blocks * ns, per, bf), chain_seconds(per, wave_count(blocks * ns, per), link)) +
                     (ns > 1 ? kWaveFinish : 0);
    if (t < 0.98 * best.seconds) best = WavePlan{ns, blocks * ns, (double)per, t};
  }
  return best;
}

template <class AL, class BL, class Epi, bool BF>
static WaveJob<AL, BL, Epi, BF> wave_job(const typename AL::Params& a, const typename BL::Params& b, const Epi& ep, int M,
                                         int N, int K, int groups, int ns) {
  WaveJob<AL, BL, Epi, BF> j;
  j.a = a;
  j.b = b;
  j.ep = ep;
  j.M = M;
  j.N = N;
  j.K = K;
  j.kchunk = ceil_div(ceil_div(K, 16), ns) * 16;
  const int gx = ceil_div(M, kWaveTile), gy = ceil_div(N, kWaveTile);
  j.gx = make_fastdiv((uint32_t)gx);
  j.gy = make_fastdiv((uint32_t)gy);
  j.ns = make_fastdiv((uint32_t)ns);
  j.blocks = (uint32_t)(gx * gy * groups * ns);
  return j;
}
template <class J>
static int launch_job(const J& j, double flops, double bytes, hipStream_t st) {
  KernelScope ks(J::BF ? "gemm_bf16" : "gemm", flops, bytes, st);
  const int waves = wave_count(j.blocks, std::min(j.K, j.kchunk) / 16);
  const dim3 grid(j.blocks), block(64 * waves);
  if (waves == 16) hipLaunchKernelGGL((gemm_wave_kernel<16, J>), grid, block, 0, st, j);
  else if (waves == 8) hipLaunchKernelGGL((gemm_wave_kernel<8, J>), grid, block, 0, st, j);
  else hipLaunchKernelGGL((gemm_wave_kernel<4, J>), grid, block, 0, st, j);
  AX_LAUNCH_CHECK();
  return ALEXNET_OK;
}
template <class J, class K>
static int launch_jobs(const J& j, const K& k, double flops, double bytes, hipStream_t st) {
  KernelScope ks(J::BF ? "gemm_bf16" : "gemm", flops, bytes, st);
  const uint32_t blocks = j.blocks + k.blocks;
  const int waves = wave_count(blocks, std::max(std::min(j.K, j.kchunk), std::min(k.K, k.kchunk)) / 16);
  const dim3 grid(blocks), block(64 * waves);
  if (waves == 16) hipLaunchKernelGGL((gemm_wave_pair_kernel<16, J, K>), grid, block, 0, st, j, k);
  else if (waves == 8) hipLaunchKernelGGL((gemm_wave_pair_kernel<8, J, K>), grid, block, 0, st, j, k);
  else hipLaunchKernelGGL((gemm_wave_pair_kernel<4, J, K>), grid, block, 0, st, j, k);
  AX_LAUNCH_CHECK();
  return ALEXNET_OK;
}
static inline double conv_work(const ConvGeom& c) { return 2.0 * c.P() * c.Cout * c.cg() * c.k * c.k; }
static inline double conv_moved(const ConvGeom& c) {
  return 4.0 * ((double)c.in_elems() + (double)c.w_elems() + (double)c.out_elems());
}

// ------------------------------------------------------------- convolution ---
static WavePlan fwd_plan(const ConvGeom& c, bool bf) {
  const GemmDims d = fwd_dims(c);
  return wave_plan(d.M, d.N, run_mode(c) ? run_k(c) : d.K, d.groups, bf, kWaveMaxK);
}
static WavePlan bwd_data_plan(const ConvGeom& c, bool bf) {
  const GemmDims d = bwdd_dims(c);
  return wave_plan(d.M, d.N, d.K, d.groups, bf, kWaveMaxK, data_link(c));
}
static WavePlan bwd_weight_plan(const ConvGeom& c, bool bf) {
  const GemmDims d = bwdw_dims(c);
  return wave_plan(d.M, d.N, d.K, d.groups, bf, kWaveMaxPixels);
}
// what the loaders take; pointwise layers, the products of transformed ones among them, are dense and stay with the tiles
// (a step of the full net at batch 16, where they would seem to pay: 1120 us, 1160 with them here)
static bool spatial(const ConvGeom& c) { return c.k > 1 || c.stride > 1; }
static bool fwd_fits(const ConvGeom& c) {
  return spatial(c) && (run_mode(c) || c.cg() % 4 == 0) && c.k <= kWaveMaxSide && c.kf() >= kSplitMinK;
}
static bool bwd_data_fits(const ConvGeom& c) {
  return spatial(c) && c.stride == 1 && c.og() % 4 == 0 && c.k <= kWaveMaxSide && c.kb() >= kSplitMinK;
}
static bool bwd_weight_fits(const ConvGeom& c) { return spatial(c) && c.k <= kWaveMaxSide && c.P() >= kSplitMinK; }
bool wave_conv_fwd_ok(const ConvGeom& c, bool bf) {
  return fwd_fits(c) && fwd_plan(c, bf).seconds < tile_floor(tile_seconds_fwd(c, bf), bf, 18e-6, conv_bf16_stored_ok(c) ? 3e-6 : 5e-6);
}
// On its own a data gradient with long rows of weights (see data_link) is better off in tiles, slices or not: bf16, second layer
// of the full net on 2 pictures 9 | 20 us, third and fourth on 4 8 | 18 and 7 | 15, fifth on 8 8 | 20.
bool wave_conv_bwd_data_ok(const ConvGeom& c, bool bf) {
  return bwd_data_fits(c) && c.og() <= 64 && bwd_data_plan(c, bf).seconds < tile_floor(tile_seconds_bwd_data(c, bf), bf);
}
bool wave_conv_bwd_weight_ok(const ConvGeom& c, bool bf) {
  return bwd_weight_fits(c) && bwd_weight_plan(c, bf).seconds < tile_floor(tile_seconds_bwd_weight(c, bf), bf, kWeightBelow);
}
// Both gradients in one launch, where the data gradient is not sliced.  beside: large dense layers are updated meanwhile, which
// slows these kernels more than tiles.  Full net, fp32, tiles against small products by the profiler, us, and what the work alone
// comes to: fourth layer, 2, 4, 6 and 8 pictures 46 | 53 (17), 58 | 75 (30), 67 | 98 (42), 82 | 131 (55); fifth, 4, 8 and 12 50 |
// 39 (21), 70 | 57 (38), 79 | 97 (55); chains of 50 and 54 steps, second and third layer, 2 pictures 40 | 77 (33) and 51 | 91
// (19); bf16 alike.  Whole steps of 2, 4, 6, 8 and 12 pictures by the work alone | by this 695 | 696, 697 | 700, 904 | 839, 876 |
// 898, 944 | 966 us, bf16 4 and 8 689 and 692 either way.
constexpr double kWaveBeside = 1.6;
bool wave_conv_bwd_ok(const ConvGeom& c, bool bf, bool beside) {
  if (!bwd_data_fits(c) || !bwd_weight_fits(c) || c.kb() > kWaveMaxK) return false;
  const WavePlan w = bwd_weight_plan(c, bf);
  const GemmDims d = bwdd_dims(c);
  const double blocks = (double)ceil_div(d.M, kWaveTile) * ceil_div(d.N, kWaveTile) * d.groups, steps = ceil_div(d.K, 16);
  const double work = wave_seconds(w.blocks + blocks * steps / w.steps, w.steps, bf) * (beside ? kWaveBeside : 1);
  const double chain = chain_seconds(steps, wave_count(w.blocks + blocks, std::max(w.steps, steps)), data_link(c));
  return std::max(work, chain) + (w.ns > 1 ? kWaveFinish : 0) <
         tile_floor(tile_seconds_bwd_data(c, bf), bf) + tile_floor(tile_seconds_bwd_weight(c, bf), bf, kWeightBelow);
}
int wave_conv_fwd_slices(const ConvGeom& c) {
  return fwd_fits(c) ? std::max(fwd_plan(c, false).ns, fwd_plan(c, true).ns) : 1;
}
int wave_conv_bwd_data_slices(const ConvGeom& c) {
  return bwd_data_fits(c) ? std::max(bwd_data_plan(c, false).ns, bwd_data_plan(c, true).ns) : 1;
}
size_t wave_conv_bwd_weight_ws_floats(const ConvGeom& c) {
  if (!bwd_weight_fits(c)) return 0;
  const int ns = std::max(bwd_weight_plan(c, false).ns, bwd_weight_plan(c, true).ns);
  return ns > 1 ? (size_t)ns * c.w_elems() : 0;
}

// a product of one launch, or of slices that a second one adds up and finishes
template <bool BF>
static int conv_fwd(const ConvGeom& c, const float* x, const float* wf, const float* bias, int relu, float* y, uint16_t* y16,
                    float* ws, int ns, hipStream_t st) {
  const GemmDims d = fwd_dims(c);
  const double fl = conv_work(c), by = conv_moved(c);
  auto product = [&](const auto& ep) -> int {
    typedef std::decay_t<decltype(ep)> Epi;
    if (run_mode(c)) {
      const WaveRunParams b{DenseParams{wf, c.Cout, 0, c.Cout, (uint32_t)(c.w_elems() * 4)}, c.k * c.Cin, run_len(c),
                            make_fastdiv((uint32_t)run_len(c))};
      return launch_job(wave_job<WaveRunA, WaveRunB, Epi, BF>(WaveRunAParams{run_A(c, x), c.k * c.Cin}, b, ep, d.M, d.N,
                                                             run_k(c), 1, ns), fl, by, st);
    }
    DenseParams b = fwd_B(c, wf);
    b.bytes = (uint32_t)(c.w_elems() / c.groups * 4);  // of a group
    return launch_job(wave_job<WaveIm2col<IM2COL_FWD>, WaveRow, Epi, BF>(fwd_A(c, x), b, ep, d.M, d.N, d.K, d.groups, ns), fl,
                      by, st);
  };
  if (ns == 1) return product(EpiBiasAct{y, c.Cout, bias, relu, c.og(), 0, 0, y16});
  AX_TRY(product(EpiSlab{ws, (long)d.M * d.N, d.N, nullptr, 0}));
  AX_TRY(launch_slab_finish(ws, ns, d.groups, d.M, d.N, bias, relu, nullptr, y, st));
  return y16 ? launch_to_bf16(y, y16, (size_t)c.out_elems(), st) : ALEXNET_OK;
}
int launch_wave_conv_fwd(const ConvGeom& c, const float* x, const float* wf, const float* bias, int relu, float* y,
                         uint16_t* y16, float* ws, bool bf, hipStream_t st) {
  const int ns = fwd_plan(c, bf).ns;
  return bf ? conv_fwd<true>(c, x, wf, bias, relu, y, y16, ws, ns, st)
            : conv_fwd<false>(c, x, wf, bias, relu, y, y16, ws, ns, st);
}

template <bool BF, class Epi>
static auto bwd_data_job(const ConvGeom& c, const float* dy, const float* wf, const Epi& ep, int ns) {
  const GemmDims d = bwdd_dims(c);
  const WaveTapParams b{DenseParams{wf, c.og(), (long)c.kf() * c.og(), c.cg(), (uint32_t)(c.w_elems() / c.groups * 4)}, c.cg(), c.og(),
                        make_fastdiv((uint32_t)c.og())};
  return wave_job<WaveIm2col<IM2COL_T1>, WaveTapB, Epi, BF>(bwdd_A(c, dy), b, ep, d.M, d.N, d.K, d.groups, ns);
}
static EpiGate gate_of(const ConvGeom& c, const float* gate, float* dx, uint16_t* dx16) {
  return EpiGate{dx, c.Cin, gate, c.cg(), 0, 0, dx16};
}
// out: ns > 1 slices [group][slice][slab], or the result
template <bool BF>
static auto bwd_weight_job(const ConvGeom& c, const float* x, const float* dy, float* out, int ns) {
  const GemmDims d = bwdw_dims(c);
  DenseParams b = bwdw_B(c, dy);
  b.bytes -= (uint32_t)(c.Cout - c.og()) * 4u;  // what lies behind the last group's origin
  return wave_job<WaveIm2colT, WaveRow, EpiSlab, BF>(fwd_A(c, x), b,
                                                     EpiSlab{out, (long)d.M * d.N, d.N, nullptr, 0}, d.M, d.N, d.K,
                                                     d.groups, ns);
}
int add_weight_slices(const ConvGeom& c, const float* slices, int ns, float* dwf, WgradTail* tail, hipStream_t st) {
  const GemmDims d = bwdw_dims(c);
  const long slab = (long)d.M * d.N;
  if (ns == 1) return ALEXNET_OK;
  if (!tail) return launch_reduce_slabs(slices, ns, slab, d.groups, dwf, st);
  if (tail->n >= kMaxWgradJobs) {
    set_error("weight-gradient tail: more than %d stages", kMaxWgradJobs);
    return ALEXNET_EINVAL;
  }
  WgradJob j{};
  j.slices = slices;
  j.dU = dwf;
  j.slab = slab;
  j.nsplit = ns;
  j.groups36 = d.groups;  // nothing to transform: total stays 0
  wgrad_tail_add(*tail, j);
  return ALEXNET_OK;
}
int launch_wave_conv_bwd_data(const ConvGeom& c, const float* dy, const float* wf, const float* gate, float* dx,
                              uint16_t* dx16, float* ws, bool bf, hipStream_t st) {
  const double fl = conv_work(c), by = conv_moved(c);
  const int ns = bwd_data_plan(c, bf).ns;
  if (ns == 1) {
    const EpiGate ep = gate_of(c, gate, dx, dx16);
    return bf ? launch_job(bwd_data_job<true>(c, dy, wf, ep, 1), fl, by, st)
              : launch_job(bwd_data_job<false>(c, dy, wf, ep, 1), fl, by, st);
  }
  const GemmDims d = bwdd_dims(c);
  const EpiSlab ep{ws, (long)d.M * d.N, d.N, nullptr, 0};
  AX_TRY((bf ? launch_job(bwd_data_job<true>(c, dy, wf, ep, ns), fl, by, st)
             : launch_job(bwd_data_job<false>(c, dy, wf, ep, ns), fl, by, st)));
  AX_TRY(launch_slab_finish(ws, ns, d.groups, d.M, d.N, nullptr, 0, gate, dx, st));
  return dx16 ? launch_to_bf16(dx, dx16, (size_t)c.in_elems(), st) : ALEXNET_OK;
}
int launch_wave_conv_bwd_weight(const ConvGeom& c, const float* x, const float* dy, float* dwf, float* slices, bool bf,
                                hipStream_t st, WgradTail* tail) {
  const int ns = bwd_weight_plan(c, bf).ns;
  float* out = ns > 1 ? slices : dwf;
  const double fl = conv_work(c), by = conv_moved(c);
  AX_TRY((bf ? launch_job(bwd_weight_job<true>(c, x, dy, out, ns), fl, by, st)
             : launch_job(bwd_weight_job<false>(c, x, dy, out, ns), fl, by, st)));
  return add_weight_slices(c, slices, ns, dwf, tail, st);
}
int launch_wave_conv_bwd(const ConvGeom& c, const float* x, const float* dy, const float* wf, const float* gate, float* dx,
                         uint16_t* dx16, float* dwf, float* slices, bool bf, hipStream_t st, WgradTail* tail) {
  const int ns = bwd_weight_plan(c, bf).ns;
  float* out = ns > 1 ? slices : dwf;
  const double fl = 2.0 * conv_work(c), by = 2.0 * conv_moved(c);
  const EpiGate ep = gate_of(c, gate, dx, dx16);
  AX_TRY((bf ? launch_jobs(bwd_weight_job<true>(c, x, dy, out, ns), bwd_data_job<true>(c, dy, wf, ep, 1), fl, by, st)
             : launch_jobs(bwd_weight_job<false>(c, x, dy, out, ns), bwd_data_job<false>(c, dy, wf, ep, 1), fl, by, st)));
  return add_weight_slices(c, slices, ns, dwf, tail, st);
}

// ------------------------------------------------------------ dense layers ---
static double dense_steps(int M, int N, int K) {
  return (double)ceil_div(M, kWaveTile) * ceil_div(N, kWaveTile) * ceil_div(K, 16);
}
// Larger weights than an XCD's L2 are streamed from memory, which wide tiles with more loads in flight do better (batch 16
// of the full net, 4 M weights and up: 1122 us a step in tiles, 1303 here).
static bool dense_fits(int in, int out) { return (double)in * out <= 1 << 20; }
bool wave_fc_fwd_ok(int B, int in, int out, bool bf) {
  const double blocks = (double)ceil_div(B, kWaveTile) * ceil_div(out, kWaveTile);
  return in >= kSplitMinK && dense_fits(in, out) &&
         wave_seconds(blocks, ceil_div(in, 16), bf) < tile_floor(tile_seconds_dense(B, out, in, bf), bf);
}
bool wave_fc_bwd_ok(int B, int in, int out, bool bf) {
  const double most = std::max(ceil_div(B, 16), ceil_div(out, 16));  // the longer of the two reductions
  return std::min(B, out) >= kSplitMinK && dense_fits(in, out) &&
         wave_seconds((dense_steps(out, in, B) + dense_steps(B, in, out)) / most, most, bf) <
             tile_floor(tile_seconds_dense(out, in, B, bf), bf) + tile_floor(tile_seconds_dense(B, in, out, bf), bf);
}

static inline double fc_work(int B, int in, int out) { return 2.0 * B * in * (double)out; }
static inline double fc_moved(int B, int in, int out) { return 4.0 * ((double)in * out + (double)B * (in + out)); }

template <bool VEC, bool BF>
static int fc_fwd_job(int B, int in, int out, const float* x, const float* w, const FcAct& act, float* y, uint16_t* y16,
                      hipStream_t st) {
  const DenseParams a{x, in, 0, B, (uint32_t)((size_t)B * in * 4)}, b{w, in, 0, out, (uint32_t)((size_t)out * in * 4)};
  return launch_job(wave_job<WaveK<VEC>, WaveK<VEC>, EpiFcAct, BF>(a, b, EpiFcAct{y, out, act, y16}, B, out, in, 1, 1),
                    fc_work(B, in, out), fc_moved(B, in, out), st);
}
int launch_wave_fc_fwd(int B, int in, int out, const float* x, const float* w, const FcAct& act, float* y, uint16_t* y16,
                       bool bf, hipStream_t st) {
  if (in % 4) return fc_fwd_job<false, false>(B, in, out, x, w, act, y, y16, st);
  if (bf) return fc_fwd_job<true, true>(B, in, out, x, w, act, y, y16, st);
  return fc_fwd_job<true, false>(B, in, out, x, w, act, y, y16, st);
}
template <bool BF>
static auto fc_bwd_weight_job(int B, int in, int out, const float* x, const float* dy, float* dw) {
  const DenseParams a{dy, out, 0, out, (uint32_t)((size_t)B * out * 4)}, b{x, in, 0, in, (uint32_t)((size_t)B * in * 4)};
  return wave_job<WaveRow, WaveRow, EpiSlab, BF>(a, b, EpiSlab{dw, (long)out * in, in, nullptr, 0}, out, in, B, 1, 1);
}
template <bool VEC, bool BF>
static auto fc_bwd_data_job(int B, int in, int out, const float* dy, const float* w, const float* gate, float* dx,
                            uint16_t* dx16) {
  const DenseParams a{dy, out, 0, B, (uint32_t)((size_t)B * out * 4)}, b{w, in, 0, in, (uint32_t)((size_t)out * in * 4)};
  return wave_job<WaveK<VEC>, WaveRow, EpiGate, BF>(a, b, EpiGate{dx, in, gate, in, 0, 0, dx16}, B, in, out, 1, 1);
}
int launch_wave_fc_bwd(int B, int in, int out, const float* x, const float* dy, const float* w, const float* gate, float* dx,
                       uint16_t* dx16, float* dw, bool bf, hipStream_t st) {
  const double fl = 2.0 * fc_work(B, in, out), by = 2.0 * fc_moved(B, in, out);
  if (out % 4)
    return launch_jobs(fc_bwd_weight_job<false>(B, in, out, x, dy, dw),
                       fc_bwd_data_job<false, false>(B, in, out, dy, w, gate, dx, dx16), fl, by, st);
  if (bf)
    return launch_jobs(fc_bwd_weight_job<true>(B, in, out, x, dy, dw),
                       fc_bwd_data_job<true, true>(B, in, out, dy, w, gate, dx, dx16), fl, by, st);
  return launch_jobs(fc_bwd_weight_job<false>(B, in, out, x, dy, dw),
                     fc_bwd_data_job<true, false>(B, in, out, dy, w, gate, dx, dx16), fl, by, st);
}

}  // namespace ax
