// Convolution configuration table, heuristic choice and launcher; the kernel
// template is in conv_igemm_kernel.h and its instantiations are spread over
// conv_cfg_*.hip so that they compile in parallel.
#include <algorithm>

#include "conv_igemm_kernel.h"

namespace cnn {
namespace conv {
namespace {

struct ConvConfig {
    const char* name;  // "TMxTNxBK"
    int tm, tn, bk, threads;
    bool direct;
    LaunchFn launch;
};

#define CNN_CONV_ENTRY(I, WMW, WNW, FM, FN, BK, KS, ST)                                        \
    ConvConfig{#WMW "x" #WNW " waves, " #FM "x" #FN " blocks, BK " #BK ", " #KS " slab groups",      \
               WMW * FM * 32, WNW * FN * 32, BK, 64 * WMW * WNW * KS, false, &launch_c##I},

#define CNN_SPLIT_ENTRY(I, WMW, WNW, FM, FN, BK)                                                              \
    ConvConfig{"bf16 parts, " #WMW "x" #WNW " waves, " #FM "x" #FN " blocks, BK " #BK, WMW * FM * 32, WNW * FN * 32, \
               BK, 64 * WMW * WNW, false, &launch_c##I},
#define CNN_DIRECT_ENTRY(I, FM, FN, KW) \
    ConvConfig{"direct, " #FM "x" #FN " blocks, " #KW " waves", FM * 32, FN * 32, 16, 64 * KW, true, &launch_c##I},

constexpr ConvConfig kConfigs[] = {
    CNN_CONV_CONFIGS(CNN_CONV_ENTRY) CNN_SPLIT_CONFIGS(CNN_SPLIT_ENTRY) CNN_DIRECT_CONFIGS(CNN_DIRECT_ENTRY)};
constexpr int kNumConfigs = sizeof(kConfigs) / sizeof(kConfigs[0]);
constexpr int kFirstSplit = 16;  // of the configurations on bf16 parts

// The fp32 matrix-core configuration of a shape when no tuned entry exists,
// fitted by hand to measured times of configurations 0 to 15 on AlexNet's, LeNet's and CIFAR-10 quick's
// layers and the single-layer sweep shapes at batches 1 to 256 (`python
// bench.py --config-table` times them all: over those 46 shapes the
// heuristic's total came within 0.5% of always picking the fastest on the
// box it was fitted on, and 4.0-4.9% over on others).  t64: output tiles of a
// 64 x 64 tile; b128: of a 128 x 128 tile.
int fp32_config(const ConvParams& p, int G) {
    const int64_t t64 = (int64_t)ceil_div(p.M, 64) * ceil_div(p.Kg, 64) * G;
    const int64_t b128 = (int64_t)ceil_div(p.M, 128) * ceil_div(p.Kg, 128) * G;
    if (p.Kg <= 32) return 8;                                         // 32 x 128
    if (std::max(p.sh, p.sw) >= 4 && p.Kg > 64) return t64 >= 4000 ? 6 : 8;  // strided stem
    if (t64 >= 4000 && p.Kg > 64) return 4;                          // 64 x 128
    if (p.Kg > 64 && p.Kg <= 128 && b128 >= 512) return 0;           // 128 x 128
    if (p.Kg >= 256 && t64 >= 300 && t64 < 1000) return 2;           // 128 x 64
    if (t64 < 1000) return 10;                                        // 64 x 64, BK 32
    return 9;                                                         // 64 x 64, BK 16
}

// Reduction chunks for a configuration: when its output tiles would give the
// 256 compute units fewer than 1.5 workgroups each, split the reduction so
// that about 1024 workgroups run, keeping at least 8 slabs per chunk.  (On
// AlexNet at batch 16 this made conv3-conv5 25-32% faster than splitting
// only below 128 tiles into 512 workgroups; batches 1, 64 and 256 measured
// the same.)
constexpr int kSplitBelowTiles = 384, kSplitTarget = 1024;
// The direct kernels share the reduction out among a workgroup's waves already,
// so only layers of at most 64 tiles (of 32 x 32 or 32 x 64) are split further,
// with at least four 16-tap runs a wave.  512 x 14 x 14, 3x3, one image, has 112
// tiles of 32 x 32, on which two to nine chunks measured no faster than one; it
// runs on 64 of 32 x 64 in four chunks (26.7 us a call, fill and ReLU included;
// on the 112 tiles 51.7 with 4 waves and 36.6 with 8).
constexpr int kDirectSplitBelow = 64, kDirectTarget = 256;
struct Chunks {
    int splits, kchunk;
};
__attribute__((always_inline)) inline Chunks chunks_of(const ConvParams& p, const ConvConfig& c) {
    const int tiles = ceil_div(p.M, c.tn) * ceil_div(p.Kg, c.tm) * p.G;
    const int nslab = ceil_div(p.Kr, c.bk);
    int splits = 1;
    if (c.direct) {
        if (tiles <= kDirectSplitBelow)
            splits = std::max(1, std::min(ceil_div(kDirectTarget, tiles), nslab / (c.threads / 64 * 4)));
    } else if (tiles <= kSplitBelowTiles) splits = std::max(1, std::min(ceil_div(kSplitTarget, tiles), nslab / 8));
    if (splits == 1) return {1, p.Kr};
    const int kchunk = ceil_div(nslab, splits) * c.bk;
    return {ceil_div(p.Kr, kchunk), kchunk};
}
void choose_splits(ConvParams& p, const ConvConfig& c) {
    const Chunks k = chunks_of(p, c);
    p.splits = k.splits;
    p.kchunk = k.kchunk;
}

// Whether a direct kernel's tap tables (two words a tap at most) hold the chunk,
// and the filter and the image fit the packed rows and columns of kWindowAny: 15 and 16
// bits, and row 0x7fff, which marks "past the reduction", outside the image from
// the first window on.
__attribute__((always_inline)) inline bool direct_fits(const ConvParams& p, int kchunk, const ConvConfig& c) {
    if (kchunk > kDirectTableBytes / 8 || direct_table_entries(kchunk, c.threads / 64) > kDirectTableBytes / 8) return false;
    return direct_window(p) != kWindowAny || (p.R <= 0x7fff && p.S <= 0xffff && p.H <= 0x7fff - p.ph);
}

// Estimated time (us) of a call on a configuration, by which the families are
// compared: a start of `base`, then per slab the larger of the latency of one
// workgroup alone and the throughput time of those that share a compute unit,
// scaled by the way the operands are read, plus the output's bytes, plus the
// fill, the ReLU pass and the atomics of a split reduction.  Weight rows that
// are not whole 16-byte vectors are read with 32-bit loads (`odd`), and rows
// much longer than what the vector L1 keeps of them cost more per slab
// (`longer`, up to 1024 taps, by the share of the tile's rows that exist).
// The constants were fitted (least squares of the logarithms, weight on the
// configurations near a shape's fastest) to times of calls through the Python
// binding with configurations 16 to 24 and the fp32 choice on 2464 shapes:
// AlexNet's, LeNet's, CIFAR-10 quick's and the sweep's layers at batches 1 to
// 256, and random ones of 7 to 227 pixels, 3 to 512 channels, filters 1x1 to
// 11x11, strides 1 to 4 (profiles/conv_choice_times.csv).  The residuals are 8
// to 11%.
struct TimeModel {
    double base, extra, mask, out, fill, sums;  // of a family
};
constexpr TimeModel kFp32Model = {5.62, 0.464, 1.08, 0.243, 7.14, 1.12},
                    kSplitModel = {5.41, 1.55, 1.02, 0.406, 5.51, 3.09},
                    kDirectModel = {4.75, 0.303, 1.04, 0.34, 3.63, 4.54};
// A call's least time: one launch, or those of a split reduction.
constexpr double kLeastUs = 8.4, kLeastSplitUs = 14.0;
// A layer of a network has neither that nor launches for the fill and the ReLU
// of a split reduction, which other layers' kernels do.  What is left of them,
// from passes of AlexNet, LeNet and CIFAR-10 quick at 19 batch sizes with 0 to 8
// us: with 1.5 AlexNet's at 1, 4 and 16 images takes 115.8, 182.1 and 326.5 us
// and CIFAR-10 quick's at 1 and 8 images 32.8 and 35.4; with a standalone call's
// estimates 122.1, 177.3, 332.2, 41.3 and 44.8.
constexpr double kFillInNetUs = 1.5;
// Per slab of one workgroup (us): latency alone, throughput share; scales of
// the two for strided gathers; of both for the other ways to read operands.
struct SlabTime {
    int cfg;
    double latency, share, strided_latency, strided_share, odd, any, longer, longer_odd;
};
constexpr SlabTime kSlabTimes[] = {
    {0, 0.509, 0.995, 1.1, 1.07, 1.1, 1.31, 0, 0},
    {2, 0.483, 0.493, 1.1, 1.19, 1.13, 1.16, 0, 0},
    {4, 0.503, 0.487, 1.1, 1.2, 1.03, 1.24, 0, 0},
    {6, 0.569, 0.756, 1.1, 1.08, 0.98, 1.29, 0.05, 0.0427},
    {8, 0.326, 0.26, 1.29, 1.16, 0.936, 1.59, 0.0918, 0.18},
    {9, 0.495, 0.226, 1.1, 1.19, 1.1, 1.23, 0.116, 0.0801},
    {10, 0.602, 0.468, 1.36, 1.27, 1.13, 1.29, 0.0723, 0.0153},
    {16, 1.19, 0.583, 1.28, 1.24, 1.17, 1.24, 0.0398, 0.0733},
    {17, 0.654, 0.286, 1.33, 1.3, 1.24, 1.16, 0.216, 0.668},
    {18, 0.666, 0.294, 1.31, 1.25, 1.07, 1.45, 0.251, 0.369},
    {19, 0.959, 0.528, 1.38, 1.28, 1.16, 1.31, 0.035, 0.116},
    {20, 0.32, 0.149, 1.56, 1.44, 1.2, 1.32, 0.46, 0.944},
    {21, 0.572, 0.335, 1.39, 1.43, 1.22, 1.37, 0.326, 0.379},
    {22, 0.307, 0.276, 1.24, 1.24, 1.45, 1.11, 0.226, 1.04},
    {23, 0.5, 0.569, 1.25, 1.25, 1.34, 1.02, 0.146, 1.12},
    {24, 0.705, 0.593, 1.26, 1.26, 1.28, 1.15, 0.022, 0.191},
};

constexpr SlabTime slab_time(int cfg) {
    const SlabTime* t = kSlabTimes;
    while (t->cfg != cfg) ++t;
    return *t;
}

// A call evaluates ten of these: with the configuration known at compile time
// its divisions become shifts, and the ten take 95 ns (470 with a loop over the
// table).
template <int CFG>
double estimate(const ConvParams& p, const Chunks& k, bool in_net) {
    constexpr ConvConfig c = kConfigs[CFG];
    constexpr TimeModel f = c.direct ? kDirectModel : CFG >= kFirstSplit ? kSplitModel : kFp32Model;
    constexpr SlabTime t = slab_time(CFG);
    const int64_t wgs = (int64_t)ceil_div(p.M, c.tn) * ceil_div(p.Kg, c.tm) * p.G * k.splits;
    const double queue = (double)(int)ceil_div64(wgs, 256);
    int slabs = ceil_div(k.kchunk, c.bk);
    if (c.direct) slabs = ceil_div(slabs, c.threads / 64);
    const double rows = std::min(1.0, p.Kr * (1.0 / 1024)) * p.Kg / (ceil_div(p.Kg, c.tm) * c.tm);
    const double reads = p.Kr % 4 ? t.odd + t.longer_odd * rows : 1.0 + t.longer * rows;
    const bool padded = p.ph > 0 || p.pw > 0;
    const double window = !padded ? 1.0 : p.RS <= 31 ? f.mask : t.any;
    const bool strided = p.sw > 1 && (c.direct || !padded || p.RS <= 63);
    const double scale = strided && !c.direct ? 1.0 : reads * window;
    const double slab = std::max(t.latency * (strided ? t.strided_latency : 1.0),
                                 queue * t.share * (strided ? t.strided_share : 1.0)) * scale;
    const double mout = 1e-6 * ((double)p.M * p.K);
    const double us = f.base + (slabs + f.extra) * slab + 4.0 * f.out * mout;
    const double sums = k.splits > 1 ? f.sums * k.splits * mout : 0.0;
    if (in_net) return us + sums + (k.splits > 1 ? kFillInNetUs : 0.0);
    return k.splits > 1 ? std::max(kLeastSplitUs, us + f.fill + sums) : std::max(kLeastUs, us);
}
double estimate_fp32(const ConvParams& p, int cfg, bool in_net) {
    switch (cfg) {  // every choice of fp32_config
        case 0: return estimate<0>(p, chunks_of(p, kConfigs[0]), in_net);
        case 2: return estimate<2>(p, chunks_of(p, kConfigs[2]), in_net);
        case 4: return estimate<4>(p, chunks_of(p, kConfigs[4]), in_net);
        case 6: return estimate<6>(p, chunks_of(p, kConfigs[6]), in_net);
        case 8: return estimate<8>(p, chunks_of(p, kConfigs[8]), in_net);
        case 9: return estimate<9>(p, chunks_of(p, kConfigs[9]), in_net);
        default: return estimate<10>(p, chunks_of(p, kConfigs[10]), in_net);
    }
}

// The products of parts that the split kernels leave out make a sum of a single
// tap 2 to 3% less accurate than its fp32 product, so neither the choice nor the
// tuner takes them for one (from two taps on they are the more accurate).
constexpr int kLeastSplitTaps = 2;

// The configuration of a shape when no tuned entry exists: the fp32 one unless
// a split or a direct one is estimated faster by a margin that leaves out the
// shapes where the estimate's error decides: for up to five workgroups per
// compute unit, where the last ones to run weigh most, the estimated gains were
// 4% too large in the mean, beyond that 1.5% too small.  On 700 random shapes
// that were not fitted to, the choice was 1.140 times as fast as the fp32 one
// (the fastest configuration 1.167), with 12 shapes more than 3% slower than it;
// the constants fitted on 460 shapes before gave 1.127 and 36.  Without margins,
// 2824 shapes gave 1.144 and 111, with them 1.140 and 44.
constexpr double kMargin = 1.06, kMarginManyWorkgroups = 1.01;
constexpr double kMarginSplitOrDirect = 1.05;  // on top of it, for a split reduction or a direct kernel
template <int CFG>
__attribute__((always_inline)) inline void consider(const ConvParams& p, bool in_net, int* best, double* least) {
    constexpr ConvConfig c = kConfigs[CFG];
    const Chunks k = chunks_of(p, c);
    if (c.direct ? !direct_fits(p, k.kchunk, c) : p.Kr < kLeastSplitTaps) return;
    const int64_t wgs = (int64_t)ceil_div(p.M, c.tn) * ceil_div(p.Kg, c.tm) * p.G * k.splits;
    double us = estimate<CFG>(p, k, in_net) * (wgs > 5 * 256 ? kMarginManyWorkgroups : kMargin);
    if (c.direct || k.splits > 1) us *= kMarginSplitOrDirect;
    if (us < *least) {
        *least = us;
        *best = CFG;
    }
}
int heuristic_config(const ConvParams& p, int G, bool in_net) {
    int best = fp32_config(p, G);
    double least = estimate_fp32(p, best, in_net);
    if (!in_net && least <= kLeastUs) return best;  // no other is estimated below kLeastUs
#define CNN_CONSIDER(I, ...) consider<I>(p, in_net, &best, &least);
    CNN_SPLIT_CONFIGS(CNN_CONSIDER)
    CNN_DIRECT_CONFIGS(CNN_CONSIDER)
#undef CNN_CONSIDER
    return best;
}

}  // namespace
}  // namespace conv

using conv::ConvParams;
using conv::kConfigs;
using conv::kNumConfigs;
using conv::heuristic_config;
using conv::choose_splits;

int conv2d_num_configs() { return kNumConfigs; }

const char* conv2d_config_name(int i) { return (i >= 0 && i < kNumConfigs) ? kConfigs[i].name : nullptr; }

namespace {

// Parameters, configuration and reduction split of a convolution; per_launch:
// images per launch (the gather's 31-bit offsets cover fewer than 2^29 input
// elements).  cfg < 0 on entry: the heuristic's choice, for a layer of a network
// or for a call by itself.
int conv_prepare(const ConvShape& s, int* cfg, ConvParams* out, int* per_launch, bool in_net = false) {
    ConvParams& prm = *out;
    prm.C = s.C; prm.H = s.H; prm.W = s.W; prm.K = s.K; prm.R = s.R; prm.S = s.S;
    prm.P = s.P; prm.Q = s.Q;
    prm.sh = s.sh; prm.sw = s.sw; prm.ph = s.ph; prm.pw = s.pw;
    prm.Cg = s.C / s.G;
    prm.Kg = s.K / s.G;
    prm.RS = s.R * s.S;
    prm.Kr = prm.Cg * prm.RS;
    prm.HW = s.H * s.W;
    prm.PQ = s.P * s.Q;
    prm.f_rs = make_fastdiv(prm.RS);
    prm.f_s = make_fastdiv(s.S);
    prm.f_pq = make_fastdiv(prm.PQ);
    prm.f_q = make_fastdiv(s.Q);
    prm.G = s.G;
    prm.splits = 1;
    prm.kchunk = prm.Kr;
    prm.relu_x = 0;
    const int64_t wbytes = (int64_t)s.K * prm.Kr * 4;
    if (wbytes >= ((int64_t)1 << 31)) return fail(CNN_ERR_UNSUPPORTED, "conv: weights exceed 2 GiB");
    prm.wbytes = (int)wbytes;
    const int64_t img = (int64_t)s.C * prm.HW;
    *per_launch = (int)std::min<int64_t>(std::max(s.N, 1), (((int64_t)1 << 29) - 1) / img);
    if (*per_launch < 1) return fail(CNN_ERR_UNSUPPORTED, "conv: one image exceeds 2^29 elements");
    prm.M = *per_launch * prm.PQ;
    if (*cfg < 0) *cfg = heuristic_config(prm, s.G, in_net);
    if (*cfg >= kNumConfigs) return fail(CNN_ERR_UNSUPPORTED, "conv: no configuration %d", *cfg);
    // One split decision for every launch of the call (the last one may hold
    // fewer images: splitting it the same way is still correct).
    choose_splits(prm, kConfigs[*cfg]);
    if (kConfigs[*cfg].direct && !conv::direct_fits(prm, prm.kchunk, kConfigs[*cfg])) {
        *cfg = 9;  // a reduction or a filter beyond the tap tables: the 64 x 64 tiles take it
        choose_splits(prm, kConfigs[*cfg]);
    }
    return CNN_OK;
}

}  // namespace

bool conv2d_config_takes(const ConvShape& s, int c) {
    ConvParams prm;
    int per_launch, cfg = c;
    if (conv_prepare(s, &cfg, &prm, &per_launch) != CNN_OK || cfg != c) return false;
    return kConfigs[c].direct || c < conv::kFirstSplit || prm.Kr >= conv::kLeastSplitTaps;
}

int conv2d_heuristic_config(const ConvShape& s, bool in_net) {
    ConvParams prm;
    int per_launch, cfg = -1;
    return conv_prepare(s, &cfg, &prm, &per_launch, in_net) == CNN_OK ? cfg : -1;
}

ConvPlan conv2d_plan(const ConvShape& s, int cfg) {
    ConvPlan plan = {false, false, -1};
    ConvParams prm;
    int per_launch, used = cfg == -2 ? 0 : cfg;
    if (conv_prepare(s, &used, &prm, &per_launch, true) != CNN_OK) return plan;
    plan.split = cfg != -2 && prm.splits > 1;
    if (cfg == -1) plan.heuristic = used;
    plan.may_split = plan.split;
    for (int c = 0; c < kNumConfigs && !plan.may_split; ++c) plan.may_split = conv::chunks_of(prm, kConfigs[c]).splits > 1;
    return plan;
}

int launch_conv2d(const ConvShape& s, const float* x, const float* w, const float* bias, int relu,
                  float* y, hipStream_t st, int cfg, const ConvOpts* opt) {
    if (opt && opt->relu_left) *opt->relu_left = false;
    if (s.N == 0) return CNN_OK;
    ConvParams prm;
    int per_launch;
    int rc = conv_prepare(s, &cfg, &prm, &per_launch, opt != nullptr);
    if (rc != CNN_OK) return rc;
    prm.w = w;
    prm.bias = bias;
    prm.relu = relu;
    prm.relu_x = opt && opt->relu_in;
    const bool vec_w = (prm.Kr % 4 == 0) && ((reinterpret_cast<uintptr_t>(w) & 15) == 0);
    const int64_t img = (int64_t)s.C * prm.HW;
    const int64_t total = (int64_t)s.N * s.K * prm.PQ;
    if (prm.splits > 1 && !(opt && opt->prefilled)) {  // y[n][k][pq] = bias[k]: the sums' start
        const BiasFill fill = make_bias_fill(y, bias, s.N, s.K, prm.PQ);
        rc = launch_bias_fills(&fill, 1, st);
        if (rc != CNN_OK) return rc;
    }
    for (int n0 = 0; n0 < s.N; n0 += per_launch) {
        const int nb = std::min(per_launch, s.N - n0);
        prm.x = x + (size_t)n0 * img;
        prm.y = y + (size_t)n0 * s.K * prm.PQ;
        prm.M = nb * prm.PQ;
        prm.xbytes = (int)(nb * img * 4);
        rc = kConfigs[cfg].launch(prm, vec_w, st);
        if (rc != CNN_OK) return rc;
    }
    if (prm.splits > 1 && relu) {
        if (opt && opt->relu_left) {  // the consumer applies it
            *opt->relu_left = true;
            return CNN_OK;
        }
        return launch_relu(y, y, total, st);
    }
    return CNN_OK;
}

}  // namespace cnn
