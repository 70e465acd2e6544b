// C ABI of the ECO library (see include/eco.h): argument validation, derivation of the fp32 step
// constants, launch plans (device tables mapping tiles to tensors) and kernel dispatch.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "../../include/eco.h"
#include "eco_internal.hpp"

namespace {

thread_local std::string g_last_error;
// launch tuning (eco_set_option): read by every eco_step, possibly from other host threads
std::atomic<int64_t> g_wgs_per_cu{0};        // 0 = default
std::atomic<int64_t> g_max_launch_threads{-1};   // -1 = the runtime's limit; smaller values make the step launch in chunks
std::atomic<int64_t> g_lds_bytes{-1};        // -1 = default; dynamic LDS per workgroup of the step kernel (occupancy limiter)
std::atomic<int64_t> g_lds_bytes_wave{-1};   // -1 = default; the same per wave of the wide-group and tensor-wise kernels

eco_status_t fail(eco_status_t st, const char *fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return st;
}

eco_status_t fail_hip(hipError_t e, const char *what) {
  return fail(ECO_EHIP, "%s: %s", what, hipGetErrorString(e));
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// hparams.block_size is the default scale group of a plan: a power of two in [32, 512] (tensors may
// override it with their own group_size)
eco_status_t check_block_size(uint32_t bs) {
  if (bs == 0) return fail(ECO_EINVAL, "block_size must be positive");
  const int s = eco::log2_exact(bs);
  if (s < 5 || s > 9) return fail(ECO_EUNSUPPORTED, "block_size %u: supported sizes are 32, 64, 128, 256, 512", bs);
  return ECO_OK;
}

bool is_dtype(int32_t d) { return d == ECO_DT_FP32 || d == ECO_DT_BF16; }

void derive_constants(const eco_hparams_t *hp, eco_constants_t *c);

// Validation of everything eco_step reads from the hyper-parameters.
eco_status_t check_hparams(const eco_hparams_t *hp) {
  if (!hp) return fail(ECO_EINVAL, "hyper-parameters: null pointer");
  if (hp->opt != ECO_OPT_ADAM && hp->opt != ECO_OPT_SGDM) return fail(ECO_EINVAL, "opt %d: unknown optimizer", hp->opt);
  if (hp->round != ECO_ROUND_SR && hp->round != ECO_ROUND_RTN) return fail(ECO_EINVAL, "round %d: unknown rounding", hp->round);
  if (hp->mode < ECO_MODE_NAIVE || hp->mode > ECO_MODE_MASTER) return fail(ECO_EINVAL, "mode %d: unknown mode", hp->mode);
  if (hp->mode == ECO_MODE_EXACT && hp->opt != ECO_OPT_SGDM)
    return fail(ECO_EUNSUPPORTED, "exact stored-error injection is defined for SGDM only");
  if (!is_dtype(hp->state_dtype) || !is_dtype(hp->scale_dtype)) return fail(ECO_EINVAL, "unknown state or scale dtype");
  if (hp->step == 0) return fail(ECO_EINVAL, "step is 1-based: step == 0 has no bias correction");
  if (!std::isfinite(hp->lr) || hp->lr < 0.0) return fail(ECO_EINVAL, "lr must be finite and >= 0");
  if (!std::isfinite(hp->weight_decay) || hp->weight_decay < 0.0) return fail(ECO_EINVAL, "weight_decay must be finite and >= 0");
  if (!(hp->beta1 >= 0.0 && hp->beta1 < 1.0)) return fail(ECO_EINVAL, "beta1 must lie in [0, 1)");
  if (hp->mode == ECO_MODE_ECO || hp->mode == ECO_MODE_EXACT) {
    // the injection strength divides by the learning rate and by beta (Eq. alpha; Alg. 3 line 5; Eq. im_inject)
    if (!(hp->lr > 0.0)) return fail(ECO_EINVAL, "error injection needs lr > 0");
    if (!(hp->beta1 > 0.0)) return fail(ECO_EINVAL, "error injection needs beta1 in (0, 1)");
  }
  if (hp->opt == ECO_OPT_ADAM) {
    if (!(hp->beta2 >= 0.0 && hp->beta2 < 1.0)) return fail(ECO_EINVAL, "beta2 must lie in [0, 1)");
    if (!std::isfinite(hp->eps) || hp->eps < 0.0) return fail(ECO_EINVAL, "eps must be finite and >= 0");
  }
  // valid doubles can still leave the fp32 range once combined (a tiny lr makes the injection strength
  // (1/lr)(1 - 1/beta) overflow): the step would then write non-finite state
  eco_constants_t c;
  derive_constants(hp, &c);
  const float all[] = {c.b1, c.omb1, c.b2, c.omb2, c.rbc2, c.c1, c.eps, c.kappa, c.lr, c.alpha, c.wd, c.inv_lr, c.inv_lr_beta};
  for (float x : all)
    if (!std::isfinite(x)) return fail(ECO_EINVAL, "a step constant derived from lr, the betas and the step index is not finite in fp32");
  return ECO_OK;
}

void derive_constants(const eco_hparams_t *hp, eco_constants_t *c) {
  const double k = static_cast<double>(hp->step);
  const double bc1 = 1.0 - std::pow(hp->beta1, k);
  const double bc2 = 1.0 - std::pow(hp->beta2, k);
  std::memset(c, 0, sizeof *c);
  c->b1 = static_cast<float>(hp->beta1);
  c->omb1 = static_cast<float>(1.0 - hp->beta1);
  c->b2 = static_cast<float>(hp->beta2);
  c->omb2 = static_cast<float>(1.0 - hp->beta2);
  c->rbc2 = static_cast<float>(1.0 / bc2);
  c->c1 = static_cast<float>(hp->lr / bc1);
  c->eps = static_cast<float>(hp->eps);
  c->lr = static_cast<float>(hp->lr);
  c->wd = static_cast<float>(hp->lr * hp->weight_decay);
  if (hp->mode == ECO_MODE_ECO) {
    c->kappa = static_cast<float>((bc1 / hp->lr) * (1.0 - 1.0 / hp->beta1));
    c->alpha = static_cast<float>((1.0 / hp->lr) * (1.0 - 1.0 / hp->beta1));
  }
  if (hp->mode == ECO_MODE_EXACT) {
    c->inv_lr = static_cast<float>(1.0 / hp->lr);
    c->inv_lr_beta = static_cast<float>(1.0 / (hp->lr * hp->beta1));
  }
}

struct Lists {                           // the launch lists of one storage format
  std::vector<uint32_t> tile;            // block-scaled: one entry per full tile
  std::vector<uint32_t> extra;           // one-wave units that ride along (ragged tails, short rows, unquantized tensors)
  std::vector<uint32_t> wide[eco::MAX_WIDE_WAVES + 1];   // wide groups, by waves per unit: one entry per unit
  std::vector<uint32_t> tw_tile;         // tensor-wise: one entry per tile (full or partial)
  std::vector<uint32_t> tw_tensor;       // tensor-wise: the tensors
  std::vector<uint32_t> slab;            // tensor-wise in one pass: one entry per slab
  std::vector<uint32_t> resident;        // tensor-wise in one pass: the tensors
  size_t off_tile = 0, off_extra = 0, off_wide[eco::MAX_WIDE_WAVES + 1] = {0}, off_tw_tile = 0, off_tw_tensor = 0, off_slots = 0,
         off_tile_max = 0, off_slab = 0, off_resident = 0, off_tail_max = 0, off_slab_max = 0, off_counts = 0, off_deferred = 0;
  uint64_t tensors = 0, most_tw_tiles = 0, tails = 0;
  struct WideLoad { uint64_t idle, elements, off_lines; };   // of a wide list: units that leave lanes idle; elements (0: the one-wave units'); those
                                                         // whose waves start off the lines of memory (0: of the full tiles as well)
  WideLoad load[eco::MAX_WIDE_WAVES + 2] = {};           // the last: long tensors with one scale
  std::vector<uint32_t> one;             // all but the tensor-wise tensors as one launch, where that is the better way: workgroup -> tensor
  size_t off_one = 0;
  unsigned one_waves = 1;
  eco::StepLaunch launch = {};           // what the step launches, but for the scalars of a call
  std::vector<uint32_t> &list(int l) {
    return l == eco::LIST_TILE ? tile : l == eco::LIST_EXTRA ? extra : l == eco::LIST_TW_TILES ? tw_tile : l == eco::LIST_RESIDENT ? slab : wide[l - eco::LIST_WIDE1 + 1];
  }
};

// Unquantized tensors of up to this many 512-element tiles together are one-wave units in the launch of a quantized
// format; more of them get the kernel that is compiled for them alone.  A launch costs 5-6 us, what 20 MB take; beyond a
// few thousand tiles the unguarded accesses of that kernel are worth more.
constexpr uint64_t RIDE_ALONG_TILES = 8192;
constexpr uint64_t RIDE_ALONG_WAVES = 65536;   // largest wide-group launch that takes them, see home_of_extra

// A step of at most this many elements that would be several launches is one launch of the list kernel instead.
constexpr uint64_t SMALL_ELEMENTS = 1ull << 23;

// How much of a step's arrays comes from HBM and not from the 256 MB cache before it, by the bytes of the arrays, each
// counted once: the caps on resident waves were measured against none over 1 to 256 M elements, and the two met between
// 340 and 420 MB where the traffic in flight is little (bf16 state), between 60 and 120 MB elsewhere.
struct HbmBound {
  bool half, fully;
  explicit HbmBound(uint64_t bytes) : half(bytes >= 96000000), fully(bytes >= 384000000) {}
};

// Bytes of all arrays of a list.  From HbmBound::half on the step groups rows in its own way (see step_geometry); in shorter
// steps the exact bundles, which leave most rows in few launches, are the better way (3.5 M elements in rows of 1024 and of 768, SGDM
// with a stored error: 6.0 us in one launch, 6.8 in two).
uint64_t bytes_of(const eco_tensor_t *tensors, size_t n, const eco::StateLayout &l) {
  uint64_t sum = 0;
  for (size_t i = 0; i < n; ++i) sum += eco::array_bytes(tensors[i].numel, tensors[i].fmt, l);
  return sum;
}

// The step's own grouping of rows has a launch for each size of workgroup, which may be more of them than the other grouping's: 4-6 us
// that it has to make up for (us, other / own, with a launch more: 16.9 M elements in rows of 4096, 1024 and an odd number of 768, FP8 with bf16
// state 41.2 / 45.8; rows of 768, 2304 and 576, 11 M, FP8 60.6 / 66.3; INT4 SGDM 39 M in rows of 1024, 768 and 1816 102.9 / 109.1; 160 M in rows of
// 576 and 1024, INT4 with bf16 state 550 / 475).  So from 384 MB on, and below where it takes no launch more.
bool own_grouping_pays(uint64_t bytes, const uint32_t (&own_sizes)[4], const uint32_t (&sizes)[4]) {
  int more = 0;
  for (int f = 0; f < 4; ++f) more += __builtin_popcount(own_sizes[f]) - __builtin_popcount(sizes[f]);
  return HbmBound(bytes).fully || more <= 0;
}

int num_compute_units() {
  int dev = 0, cus = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 256;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus <= 0) return 256;
  return cus;
}

// Resident waves per compute unit at which the full-tile step kernel measured fastest on MI355X, by bytes
// moved per 512-element tile: HBM delivers most with a certain amount of tile traffic in flight per compute unit, and
// more waves than that only add latency.  bf16 state, Adam (us, without a cap -> with it): INT4, 1.39 G elements, 2689 ->
// 2470 at 21 waves (2558 at 18, 2655 at 25); FP8, 0.42 G elements, 885 -> 824 at 18 (857 at 21, 855 at 16), with master weights 1423 -> 1310 at 12 (1381 at 16).
// Unquantized weights (22 B/parameter with fp32 state, 14 with bf16), 148 M elements: 614 -> 561 us, 374 -> 337.
// That holds for arrays that come from HBM (see HbmBound): where a step finds them in the cache before it, a cap costs up
// to 24 % (bf16 state, us, without / with: FP8 4 M elements 9.3 / 10.4, 32 M 61.1 / 60.3, 64 M 142 / 137; INT4 32 M 56.2 / 56.3,
// 48 M 85.0 / 88.2, 64 M 129.4 / 127.5; master weights 4 M 14.0 / 15.7, 32 M 105.1 / 107.7, 64 M 226 / 213; unquantized 4 M 8.6 / 10.4,
// 16 M 38.9 / 37.8).  The caps of fp32 state as well, since waves take
// whole lines (see exchange_chunks; us, with / without): Adam 40 MB 15.2 / 13.4, 120 MB 37.0 / 35.6 (35.2 at 20 waves), master weights 40 MB 15.2 /
// 13.1, 120 MB 35.0 / 32.1, 240 MB 65.6 / 66.2, SGDM 14.4 / 12.2, 32.8 / 31.9, 62.6 / 61.8, with a stored error 13.5 / 11.5, 33.9 / 32.9, 64.6 / 63.2,
// with master weights 12.7 / 10.2, 33.3 / 32.0, 64.1 / 60.7.  Adam's of 20 waves against none: 16 to 24 M elements 0.5 to 1.7 % less time
// (17 M 54.2 / 54.6, 21 M 67.5 / 68.2, 23 M 74.0 / 75.2).  Caps of 28 waves are worth nothing anywhere (28 / none: 1 M 5.25 / 5.27, 2 M 6.98 / 7.01, rows
// of 2048 5.44 / 5.43, 7.45 / 7.45; those of the wide groups 290 MB of master weights 85.3 / 85.3, 85.7 / 85.6, 79.1 / 79.2, bf16 state at 390 and
// 430 MB 97.5 / 97.1, 116.8 / 116.2, INT4 99.9 / 99.3, 115.8 / 113.0).
int default_waves(const eco::KernelVariant &kv, const HbmBound &hbm) {
  if (kv.fmt == eco::FMT_BF16_PLAIN || kv.fmt == eco::FMT_FP32_ID) {
    if (kv.state_bf16) return (eco::algo_is_adam(kv.algo) ? hbm.half : hbm.fully) ? 13 : 0;
    return hbm.half ? 12 : 0;
  }
  if (kv.state_bf16) {
    if (!hbm.fully) return 0;
    if (kv.algo == eco::ALGO_ADAM) return kv.fmt == eco::FMT_INT4 ? 21 : 18;
    return kv.algo == eco::ALGO_ADAM_MASTER ? 12 : 0;
  }
  switch (kv.algo) {
    case eco::ALGO_ADAM: return hbm.fully ? 12 : hbm.half ? 20 : 0;           // 20.1 B/parameter
    case eco::ALGO_ADAM_MASTER: return hbm.fully ? 8 : 0;    // 27.0
    case eco::ALGO_SGDM: return hbm.fully ? 14 : 0;          // 12.1
    case eco::ALGO_SGDM_MASTER: return hbm.fully ? 8 : 0;    // 19.0
    default: return hbm.fully ? 11 : 0;                      // SGDM with a stored error: 20.1
  }
}

// The same for launches that pass the caches by.  Adam with fp32 state wants more waves as long as part of the arrays is still in the cache (us,
// 12 / 20 waves: 29 M elements 117 / 112, 54 M 175 / 173, 137 M 439 / 438, 870 M 2734 / 2857).  2.8 GB of traffic, default_waves' / this: SGDM 430 /
// 421, with a stored error 442 / 430, with master weights 453 / 436.
int streaming_waves(const eco::KernelVariant &kv, uint64_t bytes) {
  if (kv.fmt == eco::FMT_BF16_PLAIN || kv.fmt == eco::FMT_FP32_ID || kv.state_bf16) return default_waves(kv, HbmBound(UINT64_MAX));
  switch (kv.algo) {
    case eco::ALGO_ADAM: return bytes < 600000000 ? 20 : 12;
    case eco::ALGO_ADAM_MASTER: return 8;
    case eco::ALGO_SGDM: return 16;
    case eco::ALGO_SGDM_MASTER: return 13;
    default: return 14;
  }
}

// The two tensor-wise passes over 210 M elements (us): Adam, fp32 state 1119 at 16 waves (1176 without a cap); INT4 with
// bf16 state 623 at 21 (645); SGDM 676 at 18 (703).  The last two for arrays from HBM only (one tensor of 4.7 M elements:
// SGDM 22.6 without a cap, 24.8 with it).
// Past the caches INT4 572 at 21 and 555 at 25.
int tensorwise_waves(const eco::KernelVariant &kv, const HbmBound &hbm, bool streamed) {
  if (kv.algo == eco::ALGO_ADAM && !kv.state_bf16) return 16;
  if (!hbm.fully) return 0;
  if (kv.algo == eco::ALGO_ADAM) return streamed ? 25 : 21;
  return kv.algo == eco::ALGO_SGDM && !kv.state_bf16 ? 18 : 0;
}

// A cap is expressed as a dynamic-LDS request the kernels never touch (160 KB of LDS per compute unit).
uint32_t lds_for_waves(int waves, int granule) {
  return waves > 0 ? static_cast<uint32_t>(163840 / waves / granule * granule) : 0u;
}

// Most threads of a full-tile launch.  Default: no limit but the runtime's, one workgroup per tile.  The hardware
// dispatcher then hands out tiles in address order, which keeps the set of DRAM pages in flight compact; grid-stride
// loops over a resident grid measured 10-15 % slower on MI355X.  Option 0 caps it to a resident grid, in pieces.
uint64_t tile_threads(uint64_t most, int cus) {
  const int64_t wgs_per_cu = g_wgs_per_cu.load(std::memory_order_relaxed);
  if (wgs_per_cu <= 0) return most;
  return std::min<uint64_t>(most, static_cast<uint64_t>(cus) * static_cast<uint64_t>(wgs_per_cu) * eco::WG_THREADS);
}

// Validation of one tensor descriptor against the layout part of the hyper-parameters; on success *gsz is the
// tensor's scale group and *cls its class (eco::GROUP_*).
eco_status_t check_tensor(const eco_tensor_t &t, size_t i, const eco_hparams_t *layout, uint64_t *gsz, int *cls) {
  const bool needs_aux = layout->mode == ECO_MODE_EXACT || layout->mode == ECO_MODE_MASTER;
  if (t.fmt < ECO_FMT_FP8_E4M3 || t.fmt > ECO_FMT_FP32_IDENTITY) return fail(ECO_EINVAL, "tensor %zu: unknown format %d", i, t.fmt);
  if (t.numel == 0) return fail(ECO_EINVAL, "tensor %zu: numel == 0", i);
  const bool quantized = t.fmt == ECO_FMT_FP8_E4M3 || t.fmt == ECO_FMT_INT4;
  if (!t.weights || !t.grad || !t.m) return fail(ECO_EINVAL, "tensor %zu: null weights, grad or m", i);
  if (quantized && !t.scales) return fail(ECO_EINVAL, "tensor %zu: quantized format needs scales", i);
  if (layout->opt == ECO_OPT_ADAM && !t.v) return fail(ECO_EINVAL, "tensor %zu: Adam needs v", i);
  if (quantized && needs_aux && !t.aux) return fail(ECO_EINVAL, "tensor %zu: this mode needs the aux buffer", i);
  if (!aligned16(t.weights) || !aligned16(t.grad) || !aligned16(t.m) || (quantized && !aligned16(t.scales)) ||
      (layout->opt == ECO_OPT_ADAM && !aligned16(t.v)) || (quantized && needs_aux && !aligned16(t.aux)))
    return fail(ECO_EALIGN, "tensor %zu: every data pointer must be 16-byte aligned", i);
  *gsz = t.group_size ? t.group_size : layout->block_size;
  *cls = quantized ? eco::classify_group(*gsz, t.numel) : eco::GROUP_BLOCK;
  if (*cls == eco::GROUP_UNSUPPORTED)
    return fail(ECO_EUNSUPPORTED, "tensor %zu: scale group of %llu elements: supported are powers of two in [32, 512], "
                "multiples of 8 up to 8192, and the whole tensor", i, (unsigned long long)*gsz);
  return ECO_OK;
}

// The layout part of the hyper-parameters (what eco_plan_create reads).
eco_status_t check_layout(const eco_hparams_t *layout) {
  if (!layout) return fail(ECO_EINVAL, "plan: null layout");
  if (layout->opt != ECO_OPT_ADAM && layout->opt != ECO_OPT_SGDM) return fail(ECO_EINVAL, "opt %d: unknown optimizer", layout->opt);
  if (!is_dtype(layout->state_dtype) || !is_dtype(layout->scale_dtype)) return fail(ECO_EINVAL, "unknown state or scale dtype");
  if (layout->mode < ECO_MODE_NAIVE || layout->mode > ECO_MODE_MASTER) return fail(ECO_EINVAL, "mode %d: unknown mode", layout->mode);
  if (layout->mode == ECO_MODE_EXACT && layout->opt != ECO_OPT_SGDM)
    return fail(ECO_EUNSUPPORTED, "exact stored-error injection is defined for SGDM only");
  return check_block_size(layout->block_size);
}

eco::StateLayout state_layout(const eco_hparams_t *layout) {
  return {layout->opt == ECO_OPT_ADAM, layout->state_dtype == ECO_DT_BF16, layout->mode == ECO_MODE_EXACT || layout->mode == ECO_MODE_MASTER,
          layout->mode == ECO_MODE_MASTER};
}

// The kernel variant of a step with these hyper-parameters on tensors of format f.
eco::KernelVariant variant_for(const eco_hparams_t *hp, int f) {
  eco::KernelVariant kv;
  kv.fmt = f;
  kv.state_bf16 = hp->state_dtype == ECO_DT_BF16;
  kv.scale_bf16 = hp->scale_dtype == ECO_DT_BF16;
  if (hp->mode == ECO_MODE_MASTER) kv.algo = hp->opt == ECO_OPT_ADAM ? eco::ALGO_ADAM_MASTER : eco::ALGO_SGDM_MASTER;
  else if (hp->mode == ECO_MODE_EXACT) kv.algo = eco::ALGO_SGDM_EXACT;
  else kv.algo = hp->opt == ECO_OPT_ADAM ? eco::ALGO_ADAM : eco::ALGO_SGDM;
  kv.round = hp->round;
  return kv;
}

// Whether the waves that step a tensor start off the 128-byte lines of its arrays: its units are no multiple of 64 elements, the line of a
// bf16 array, or an array does not begin on a line.  Of the arrays that the step uses: the others' pointers may be anything.
bool off_lines(const eco_tensor_t &t, const eco::Placement &p, const eco::StateLayout &l) {
  uintptr_t arrays = reinterpret_cast<uintptr_t>(t.weights) | reinterpret_cast<uintptr_t>(t.grad) | reinterpret_cast<uintptr_t>(t.m);
  if (l.adam) arrays |= reinterpret_cast<uintptr_t>(t.v);
  if (l.aux && (t.fmt == ECO_FMT_FP8_E4M3 || t.fmt == ECO_FMT_INT4)) arrays |= reinterpret_cast<uintptr_t>(t.aux);
  const bool units_of_rows = p.kind == eco::UNIT_WIDE || p.kind == eco::UNIT_ROWS || p.kind == eco::UNIT_ROW;
  return (arrays & 127) != 0 || (units_of_rows && p.units > 1 && p.rows * p.group % 64 != 0);
}

// Which launches of a step pass the caches by (CACHED and the others beside it in the kernels say what that is worth), a bit each: 0 the
// full-tile one, n the wide groups of n waves, STREAM_TENSORWISE the others.  Arrays that the 256 MB cache before HBM still holds from the step before lose by it, and so do
// waves that start off the lines of memory, whose instructions then write parts of two (us, us usual / streamed) -- by bytes of the arrays, groups
// of 128: fp32 state, Adam 250 MB 71 / 74, 280 89 / 82, 340 103 / 99, master weights 69 / 74, 91 / 82, 107 / 97, SGDM 65 / 69, 82 / 77; bf16
// state, INT4, Adam 310 MB 82 / 83, 340 90 / 90, 420 99 / 97, 640 187 / 168, SGDM (FP8) 310 75 / 78, 340 84 / 85, 420 101 / 95.  Rows of 1.6 GB, fp32
// state: 1120 (pairs: 35 lines) 491 / 451, 2016 517 / 507, 544 532 / 555, 1000 527 / 654, 6944 545 / 554; bf16 state 1120 528 / 620, 320 590 / 576.
// The line of fp32 state among the forms, 285 / 300 / 320 / 340 MB, streamed in hundredths of usual: Adam groups of 128 104 / 105 / 101 / 98, rows of
// 1024 100 / 99 / 94 / 89, 1088 106 / 110 / 101 / 94, 192 104 / 107 / 106 / 103; with master weights 128 98 / 105 / 103 / 94, rows of 1024 109 / 108 / 95 / 90;
// SGDM 128 102 / 103 / 103 / 98, rows of 1024 96 / 97 / 96 / 91.  All of these are of steps back to back on the same arrays.  What a training loop does
// between two steps takes the place of the arrays in the cache, and the two would meet at less there; no rule here is measured for that.
constexpr uint64_t stream_from(bool f32) { return f32 ? 310000000 : 384000000; }
uint32_t stream_launches(uint64_t bytes, bool f32, uint64_t tiles, const Lists::WideLoad (&load)[eco::MAX_WIDE_WAVES + 2]) {
  if (bytes < stream_from(f32)) return 0;
  uint32_t launches = load[0].off_lines * 8 <= load[0].elements + tiles * eco::TILE_ELEMS ? 1 : 0;
  for (int nw = 1; nw <= eco::STREAM_TENSORWISE; ++nw) launches |= (load[nw].off_lines * 8 <= load[nw].elements ? 1u : 0u) << nw;
  return launches;
}

// Which launch the one-wave units of a format ride in: the full-tile one (0) where there is one, they are many or every
// wide-group launch is long, else the wide-group one with the most units.  Riding in a wide-group launch costs 3.6 % of
// it, a launch of their own 5 us: the two meet at about 35 million elements.
int home_of_extra(uint64_t tiles, uint64_t extra, const uint32_t (&num_wide)[eco::MAX_WIDE_WAVES + 1]) {
  int best = 0;
  uint64_t most = 0;
  if (tiles || extra > RIDE_ALONG_TILES) return 0;
  for (int nw = 1; nw <= eco::MAX_WIDE_WAVES; ++nw) {
    const uint64_t waves = static_cast<uint64_t>(num_wide[nw]) * nw;
    if (waves > most && waves <= RIDE_ALONG_WAVES) { best = nw; most = waves; }
  }
  return best;
}

// What the lists decide about their launches: which pass the caches by, the caps on resident waves, where the one-wave units ride.  A plan
// has it worked out once (host time of a step of one matrix in C, us: on every step 3.16, so 3.13).
typedef Lists::WideLoad WideLoads[eco::MAX_WIDE_WAVES + 2];
void choose_launches(const eco::KernelVariant &kv, const WideLoads &load, uint64_t bytes, eco::StepLaunch *sl) {
  const eco::StepArgs *a = &sl->args;
  const HbmBound hbm(bytes);
  sl->stream = stream_launches(bytes, !kv.state_bf16, a->num_tiles, load);
  const int waves = default_waves(kv, hbm), tile_waves = sl->stream & 1u ? streaming_waves(kv, bytes) : waves;
  // a launch of one-wave units beside few tiles does not have the tiles' cap, which counts on every lane; short rows alone have
  // one of their own
  const bool units = (kv.fmt == eco::FMT_FP8 || kv.fmt == eco::FMT_INT4) && a->num_extra > a->num_tiles / 8;
  const unsigned resident = units && !a->num_tiles && load[0].elements ? eco::unit_workgroups(kv, bytes, a->num_extra, load[0].elements, sl->stream & 1u) : 0;
  sl->lds_bytes = units ? eco::lds_for_workgroups(resident) : lds_for_waves(tile_waves, 512);
  for (unsigned nw = 1; nw <= static_cast<unsigned>(eco::MAX_WIDE_WAVES); ++nw) {
    const uint64_t units = sl->num_wide[nw];
    if (!units) continue;
    const bool idle = load[nw].idle > units / 8, adam32 = kv.algo == eco::ALGO_ADAM && !kv.state_bf16;
    // Workgroups of 4 and 8 waves with bf16 state gain by their cap in the cache too (4 M elements 9.7 against 10.2 us); Adam with fp32 state in
    // rows with idle lanes from 96 MB on (us, with / without: rows of 1000 88 MB 28.8 / 29.5, 33 MB 12.1 / 10.7; 1800 28.4 / 29.2, 12.1 / 11.4); the
    // others from 384 MB on (master weights, rows of 1152, 300 MB 89 / 87, of 2048 120 MB 35.9 / 33.1; SGDM, rows of 1000, 315 MB 91 / 89), of rows
    // with idle lanes some later still (see wide_workgroups_idle).  Launches that pass the caches by from 450 MB on (Adam, fp32 state, rows of 2048
    // 340 MB 95 / 90, 590 MB 174 / 191, 4096 330 MB 91.7 / 88.9, 500 MB 147 / 161).
    const bool streamed = (sl->stream >> nw & 1u) != 0;
    const bool worth = streamed ? bytes >= 450000000
                                : hbm.fully || (kv.state_bf16 ? !idle && (nw == 4 || nw == 8) : hbm.half && idle && adam32);
    const unsigned k = !worth ? 0 : idle ? eco::wide_workgroups_idle(kv, bytes, nw, units, load[nw].elements, streamed)
                                         : eco::wide_workgroups(kv, nw, streamed);
    // Adam with fp32 state in full rows has the full-tile kernel's LDS per wave (8 to 12 waves for workgroups of up to 4, two workgroups
    // of larger ones): 16 waves are 3-25 % faster where the arrays lie well (rows of 2048: 467
    // against 498) but 20 % slower where memory is the slower kind (rows of 2048 and 1408, 185 M elements: 922 against 765).
    sl->lds_bytes_wide[nw] = adam32 && !idle && !streamed ? std::min(lds_for_waves(waves, 256) * nw, 65536u) : eco::lds_for_workgroups(k);
  }
  sl->lds_bytes_tw = lds_for_waves(tensorwise_waves(kv, hbm, sl->stream >> eco::STREAM_TENSORWISE & 1u), 256);
  sl->extra_in = home_of_extra(a->num_tiles, a->num_extra, sl->num_wide);
}

// The scalar part of the kernel arguments: step constants, random-stream key; and the launch options that are set.
void fill_step_scalars(const eco_hparams_t *hp, const eco_constants_t &c, eco::StepLaunch *sl) {
  eco::StepArgs *a = &sl->args;
  a->b1 = c.b1; a->omb1 = c.omb1; a->b2 = c.b2; a->omb2 = c.omb2; a->rbc2 = c.rbc2; a->c1 = c.c1; a->eps = c.eps;
  a->kappa = c.kappa; a->lr = c.lr; a->alpha = c.alpha; a->wd = c.wd; a->inv_lr = c.inv_lr; a->inv_lr_beta = c.inv_lr_beta;
  a->seed_lo = static_cast<uint32_t>(hp->seed);
  a->seed_hi = static_cast<uint32_t>(hp->seed >> 32);
  a->step_lo = static_cast<uint32_t>(hp->step);
  a->div_mid = (c.c1 >= 0x1p-40f && c.c1 <= 0x1p40f && c.eps <= 1.0f) ? 1u : 0u;
  const int64_t opt_threads = g_max_launch_threads.load(std::memory_order_relaxed);
  sl->max_launch_threads = opt_threads > 0 ? static_cast<uint64_t>(opt_threads) : eco::MAX_LAUNCH_THREADS;
  a->unit_base = 0;
  const int64_t opt_lds = g_lds_bytes.load(std::memory_order_relaxed);
  const int64_t opt_lds_wave = g_lds_bytes_wave.load(std::memory_order_relaxed);
  if (opt_lds >= 0) sl->lds_bytes = static_cast<uint32_t>(opt_lds);
  if (opt_lds_wave >= 0) {
    for (unsigned nw = 1; nw <= static_cast<unsigned>(eco::MAX_WIDE_WAVES); ++nw)
      sl->lds_bytes_wide[nw] = std::min(static_cast<uint32_t>(opt_lds_wave) * nw, 65536u);
    sl->lds_bytes_tw = static_cast<uint32_t>(opt_lds_wave);
  }
}


// ------------------------------------------------------------------------------------------------------------
// eco_step_tensors_noalloc: the plan-less step for callers that cannot allocate.  What eco_step_tensors puts
// into freshly allocated device memory -- the tensor descriptors, the tile -> tensor launch tables, and the
// abs-max slots and per-tile maxima of tensor-wise scaling -- lives in one static device array here; the tables
// are written by a small kernel from descriptors passed as kernel arguments, so nothing is copied from host
// memory either.  Every call on a GPU shares that GPU's array: calls that overlap on one GPU race.
namespace noalloc {

constexpr uint32_t MAX_TENSORS = ECO_NOALLOC_MAX_TENSORS;
constexpr uint32_t MAX_UNITS = ECO_NOALLOC_MAX_UNITS;
constexpr size_t OFF_DESCS = 0;
constexpr size_t OFF_TABLES = OFF_DESCS + sizeof(eco::TensorDesc) * MAX_TENSORS;       // launch lists, back to back
constexpr size_t OFF_SLOTS = OFF_TABLES + sizeof(uint32_t) * MAX_UNITS;                // one per tensor-wise tensor
constexpr size_t OFF_TILE_MAX = OFF_SLOTS + sizeof(uint32_t) * MAX_TENSORS;            // one per tensor-wise tile
constexpr size_t SCRATCH_BYTES = OFF_TILE_MAX + sizeof(uint32_t) * MAX_UNITS;
static_assert(OFF_TABLES % 256 == 0 && OFF_SLOTS % 256 == 0 && OFF_TILE_MAX % 256 == 0, "scratch sections stay aligned");

static __device__ __align__(256) unsigned char scratch[SCRATCH_BYTES];

// The array's device address, per device: in host code the array's name is only a handle for
// hipGetSymbolAddress, never an address a kernel could use.
constexpr int MAX_DEVICES = 32;
std::mutex g_mu;
unsigned char *g_scratch_ptr[MAX_DEVICES] = {nullptr};

eco_status_t scratch_for_current_device(unsigned char **out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return fail_hip(e, "hipGetDevice");
  if (dev < 0 || dev >= MAX_DEVICES) return fail(ECO_EUNSUPPORTED, "device %d: only devices 0..%d are supported", dev, MAX_DEVICES - 1);
  std::lock_guard<std::mutex> lock(g_mu);
  if (!g_scratch_ptr[dev]) {
    void *p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess || !p) return fail_hip(e, "hipGetSymbolAddress(scratch)");
    g_scratch_ptr[dev] = static_cast<unsigned char *>(p);
  }
  *out = g_scratch_ptr[dev];
  return ECO_OK;
}

// One launch of the table builder carries up to BUILD_CHUNK descriptors by value.
constexpr int BUILD_CHUNK = 32;
struct BuildArgs {
  eco::TensorDesc desc[BUILD_CHUNK];
  uint32_t list_pos[BUILD_CHUNK];    // index into the tables of the first of this tensor's `units` entries
  uint32_t units[BUILD_CHUNK];       // entries (tiles or groups) the tensor adds to its launch list
  uint32_t extra_pos[BUILD_CHUNK];   // index of one more entry (a ragged tail, tensor-wise tensor list), or NO_ENTRY
  uint32_t slot_pos[BUILD_CHUNK];    // the tensor's abs-max slot (tensor-wise scaling), or NO_ENTRY
  uint32_t first_index;              // descriptor index of desc[0]
  uint32_t count;
  unsigned char *scratch;
};
constexpr uint32_t NO_ENTRY = 0xFFFFFFFFu;
static_assert(sizeof(BuildArgs) <= 4096, "kernel arguments are limited to 4 KB");

constexpr int BUILD_THREADS = 256, BUILD_BLOCKS_PER_TENSOR = 32;
__global__ __launch_bounds__(BUILD_THREADS) void eco_noalloc_build_kernel(const BuildArgs a) {
  const uint32_t k = blockIdx.x;
  if (k >= a.count) return;
  const uint32_t index = a.first_index + k;
  uint32_t *tables = reinterpret_cast<uint32_t *>(a.scratch + OFF_TABLES);
  if (blockIdx.y == 0 && threadIdx.x < sizeof(eco::TensorDesc) / sizeof(uint64_t)) {
    const uint64_t *src = reinterpret_cast<const uint64_t *>(&a.desc[k]);
    reinterpret_cast<uint64_t *>(a.scratch + OFF_DESCS)[(size_t)index * (sizeof(eco::TensorDesc) / sizeof(uint64_t)) + threadIdx.x] =
        src[threadIdx.x];
  }
  if (blockIdx.y == 0 && threadIdx.x == 0 && a.extra_pos[k] != NO_ENTRY) tables[a.extra_pos[k]] = index;
  if (blockIdx.y == 0 && threadIdx.x == 0 && a.slot_pos[k] != NO_ENTRY) reinterpret_cast<uint32_t *>(a.scratch + OFF_SLOTS)[a.slot_pos[k]] = 0;
  const uint32_t pos = a.list_pos[k], n = a.units[k];
  for (uint32_t i = blockIdx.y * BUILD_THREADS + threadIdx.x; i < n; i += BUILD_BLOCKS_PER_TENSOR * BUILD_THREADS)
    tables[pos + i] = index;
}

}  // namespace noalloc

}  // namespace

struct eco_plan {
  uint32_t block_size = 0;
  int32_t state_dtype = 0, scale_dtype = 0, opt = 0, mode = 0;
  int cus = 256;
  int device = 0;    // the device that was current when the plan was created (its tables live there)
  Lists lists[4];    // indexed by eco_format_t; unquantized tensors may be in a quantized format's lists
  bool unfinished = false;               // a step has stopped between its launches: scratch may hold what it left
  eco::TensorDesc *d_descs = nullptr;
  uint32_t *d_tables = nullptr;          // all lists, back to back, then the abs-max slots and the scratch of the tensor-wise passes
};

namespace {

// The descriptor of a tensor whose units go to a list from number `first_unit` on.
eco::TensorDesc describe(const eco_tensor_t &t, const eco_hparams_t *layout, const eco::Placement &p, uint64_t first_unit) {
  eco::TensorDesc d;
  std::memset(&d, 0, sizeof d);
  d.w = t.weights; d.s = t.scales; d.g = t.grad; d.m = t.m; d.v = t.v; d.aux = t.aux;
  d.numel = t.numel;
  d.tensor_id = t.tensor_id;
  const bool plain = p.kind == eco::UNIT_PLAIN_BF16 || p.kind == eco::UNIT_PLAIN_FP32;
  d.group_size = plain ? layout->block_size : p.group;
  if (p.kind == eco::UNIT_TILES && p.list < eco::LIST_TW_TILES) d.bs_shift = static_cast<uint16_t>(eco::log2_exact(p.group));
  if (p.kind == eco::UNIT_ROW) d.bs_shift = 9;                   // reduced over the whole wave
  d.kind = static_cast<uint16_t>(p.tail ? eco::UNIT_TAIL : p.kind);
  d.slot = p.rows;
  d.first_unit = static_cast<uint32_t>(first_unit);
  return d;
}

// Scratch that a step expects empty and leaves empty, as eco_plan_create uploads it: abs-max slots, slab maxima, marks, counts.
// Only a step that stopped between its launches (ECO_EHIP) leaves it otherwise; the next one empties it first.
constexpr int RESET_THREADS = 256, RESET_BLOCKS = 64;
__global__ __launch_bounds__(RESET_THREADS) void eco_reset_scratch_kernel(uint32_t *slots, uint32_t num_slots, uint32_t *slab_max,
                                                                          uint32_t *deferred, uint32_t num_slabs, uint32_t *counts) {
  const uint32_t first = blockIdx.x * RESET_THREADS + threadIdx.x;
  for (uint32_t i = first; i < num_slots; i += RESET_BLOCKS * RESET_THREADS) slots[i] = 0;
  for (uint32_t i = first; i < num_slabs; i += RESET_BLOCKS * RESET_THREADS) { slab_max[i] = 0xFFFFFFFFu; deferred[i] = 0; }
  if (first < 2) counts[first] = 0;
}

hipError_t reset_scratch(const eco_plan &plan, hipStream_t stream) {
  for (const Lists &g : plan.lists) {
    if (g.tw_tensor.empty() && g.slab.empty()) continue;
    uint32_t *const t = plan.d_tables;
    hipLaunchKernelGGL(eco_reset_scratch_kernel, dim3(RESET_BLOCKS), dim3(RESET_THREADS), 0, stream, t + g.off_slots,
                       static_cast<uint32_t>(g.tw_tensor.size()), t + g.off_slab_max, t + g.off_deferred,
                       static_cast<uint32_t>(g.slab.size()), t + g.off_counts);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

// Which format's launches the unquantized tensors ride in: their own, or a quantized format's of the same step.
int home_of_plain(const uint64_t (&tensors)[4], const uint64_t (&entries)[4]) {
  const uint64_t plain = entries[eco::FMT_BF16_PLAIN] + entries[eco::FMT_FP32_ID];
  if (plain > RIDE_ALONG_TILES) return -1;
  if (tensors[eco::FMT_FP8]) return eco::FMT_FP8;
  if (tensors[eco::FMT_INT4]) return eco::FMT_INT4;
  return -1;
}

// One scale for a tensor of up to 8192 elements whose length is no multiple of 8: one group of a row or list launch, or, beside longer
// tensors with one scale, one more tensor of their launches.  The second is less of a launch or a launch fewer, the first
// less work: it wins from 1600 tiles and tensors on (us, in a launch of their own / along with one of 9000 elements: FP8 300 of 770
// 16.8 / 14.7, 600 16.8 / 17.1, 1200 18.3 / 23.6, 200 of 2627 17.5 / 14.6, 60 of 8001 18.6 / 15.1, 120 18.9 / 20.2, 300 of 101 16.6 / 14.7, 1500
// 17.2 / 17.8; INT4 with bf16 state 770 16.2 / 15.1, 16.3 / 16.3, 17.6 / 19.4; where norms are stepped in that launch anyway, beside two of
// 11 942, 31 of 770 19.5 / 19.0, 60 of 8001 20.9 / 19.5), and where the longer ones are stepped in one pass, which odd lengths cost a launch
// or take from one turn to two passes, unless two passes for all are a launch fewer.
constexpr uint64_t ODD_ALONG_ENTRIES = 1600;
bool short_odd(const eco_tensor_t &t, const eco_hparams_t *layout) {
  const bool quantized = t.fmt == ECO_FMT_FP8_E4M3 || t.fmt == ECO_FMT_INT4;
  return quantized && t.numel <= eco::MAX_WIDE_GROUP && t.numel % eco::ELEMS_PER_LANE != 0 &&
         eco::classify_group(t.group_size ? t.group_size : layout->block_size, t.numel) == eco::GROUP_TENSOR;
}

// A tensor in a list launch (step_list_workgroup) of workgroups of nw waves: the waves of its units, and its workgroups.
unsigned unit_waves(const eco::Placement &p) { return p.kind == eco::UNIT_WIDE ? static_cast<unsigned>(p.list - eco::LIST_WIDE1 + 1) : 1u; }
uint64_t list_workgroups(const eco::Placement &p, unsigned nw) {
  const uint64_t units = p.units + (p.tail ? 1 : 0);
  const unsigned waves = unit_waves(p), per_wg = waves == 1 ? nw : nw / waves;      // (without the divisions that can be spared)
  return per_wg == 1 ? units : (units + per_wg - 1) / per_wg;
}
eco::TensorDesc describe_in_list(const eco_tensor_t &t, const eco_hparams_t *layout, eco::Placement p, uint64_t first_wg) {
  p.tail = false;                                       // whole and partial tiles alike there
  return describe(t, layout, p, first_wg);
}

// The arguments by value of up to SMALL_TENSORS tensors.
struct SmallItem { const eco_tensor_t *t; eco::Placement p; };
void make_small(const SmallItem *items, size_t n, const eco_hparams_t *layout, eco::SmallArgs *sa, uint64_t *wgs, unsigned *waves) {
  unsigned nw = 1;
  for (size_t i = 0; i < n; ++i) nw = std::max(nw, unit_waves(items[i].p));
  uint64_t wg = 0;
  for (size_t i = 0; i < n; ++i) {
    sa->first_wg[i] = static_cast<uint32_t>(wg);
    sa->desc[i] = describe_in_list(*items[i].t, layout, items[i].p, wg);
    wg += list_workgroups(items[i].p, nw);
  }
  sa->num = static_cast<uint32_t>(n);
  *wgs = wg;
  *waves = nw;
}

}  // namespace

extern "C" {

const char *eco_status_string(int s) {
  switch (s) {
    case ECO_OK: return "ok";
    case ECO_EINVAL: return "invalid argument";
    case ECO_EALIGN: return "misaligned pointer";
    case ECO_EUNSUPPORTED: return "unsupported combination";
    case ECO_EHIP: return "HIP runtime error";
    case ECO_ENOMEM: return "out of memory";
  }
  return "unknown status";
}

const char *eco_last_error(void) { return g_last_error.c_str(); }

int eco_version(void) { return 200; }

eco_status_t eco_set_option(int32_t option, int64_t value) {
  if (option == 0) {
    if (value < 0 || value > 65536) return fail(ECO_EINVAL, "workgroups per compute unit must lie in [0, 65536]");
    g_wgs_per_cu = value;
    return ECO_OK;
  }
  if (option == 1) {
    if (value < -1 || value > 65536) return fail(ECO_EINVAL, "LDS bytes per workgroup must lie in [-1, 65536]");
    g_lds_bytes = value;
    return ECO_OK;
  }
  if (option == 2) {
    if (value < -1 || value > 32768) return fail(ECO_EINVAL, "LDS bytes per wave must lie in [-1, 32768]");
    g_lds_bytes_wave = value;
    return ECO_OK;
  }
  if (option == 3) {
    if (value != -1 && (value < 1024 || value > static_cast<int64_t>(eco::MAX_LAUNCH_THREADS)))
      return fail(ECO_EINVAL, "threads per launch must be -1 or lie in [1024, 2^32 - 1]");
    g_max_launch_threads = value;
    return ECO_OK;
  }
  return fail(ECO_EINVAL, "unknown option %d", option);
}

eco_status_t eco_step_constants(const eco_hparams_t *hp, eco_constants_t *out) {
  if (!out) return fail(ECO_EINVAL, "constants: null output");
  const eco_status_t st = check_hparams(hp);
  if (st != ECO_OK) return st;
  derive_constants(hp, out);
  return ECO_OK;
}

eco_status_t eco_plan_destroy(eco_plan_t *plan) {
  if (!plan) return ECO_OK;
  eco_status_t st = ECO_OK;
  if (plan->d_descs || plan->d_tables) {
    // steps may still be running on the plan's device: wait for that device, whichever is current
    int cur = -1;
    const bool have_cur = hipGetDevice(&cur) == hipSuccess;
    if (have_cur && cur != plan->device) (void)hipSetDevice(plan->device);
    const hipError_t e = hipDeviceSynchronize();
    if (e != hipSuccess) st = fail_hip(e, "hipDeviceSynchronize");
    if (plan->d_descs) (void)hipFree(plan->d_descs);
    if (plan->d_tables) (void)hipFree(plan->d_tables);
    if (have_cur && cur != plan->device) (void)hipSetDevice(cur);
  }
  delete plan;
  return st;
}

eco_status_t eco_plan_create(const eco_tensor_t *tensors, size_t n, const eco_hparams_t *layout, eco_plan_t **out) {
  if (!out) return fail(ECO_EINVAL, "plan: null output pointer");
  *out = nullptr;
  if (!tensors || n == 0) return fail(ECO_EINVAL, "plan: empty tensor list");
  eco_status_t st = check_layout(layout);
  if (st != ECO_OK) return st;

  eco_plan *plan = new (std::nothrow) eco_plan;
  if (!plan) return fail(ECO_ENOMEM, "plan: host allocation failed");
  plan->block_size = layout->block_size;
  plan->state_dtype = layout->state_dtype;
  plan->scale_dtype = layout->scale_dtype;
  plan->opt = layout->opt;
  plan->mode = layout->mode;

  hipError_t e = hipSuccess;
  uint64_t bytes = 0;
  std::vector<eco::TensorDesc> descs;
  std::vector<uint32_t> host;
  try {
    // validation and placement; how much there is of every list
    std::vector<eco::Placement> place(n);
    const eco::StateLayout state = state_layout(layout);
    uint64_t tensors_of[4] = {0}, entries_of[4] = {0}, list_entries[4][eco::LIST_COUNT] = {{0}};
    bytes = bytes_of(tensors, n, state);           // of all arrays
    eco::StepRows rows = {state, HbmBound(bytes).half};
    uint32_t own_sizes[4] = {0}, sizes[4] = {0};          // of workgroups, a bit each: with the step's own grouping of rows, and without
    for (size_t i = 0; i < n && st == ECO_OK; ++i) {
      const eco_tensor_t &t = tensors[i];
      uint64_t gsz = 0;
      int cls = 0;
      st = check_tensor(t, i, layout, &gsz, &cls);
      if (st != ECO_OK) break;
      const bool quantized = t.fmt == ECO_FMT_FP8_E4M3 || t.fmt == ECO_FMT_INT4;
      place[i] = eco::place_tensor(t.numel, gsz, cls, quantized, t.fmt, eco::TILE_ELEMS, 0, &rows);
      if (rows.own_rows && place[i].kind == eco::UNIT_WIDE) {
        own_sizes[t.fmt] |= 1u << (place[i].list - eco::LIST_WIDE1);
        sizes[t.fmt] |= 1u << (eco::wide_geometry(t.numel, place[i].group).waves - 1);
      }
      tensors_of[t.fmt] += 1;
      entries_of[t.fmt] += place[i].entries;
      uint64_t &in_list = list_entries[t.fmt][place[i].list];
      in_list += place[i].entries;
      if (in_list > 0x7FFFFFF0ull) st = fail(ECO_EUNSUPPORTED, "plan: more than 2^31 tiles in one launch");
    }
    if (st != ECO_OK) { delete plan; return st; }
    if (rows.own_rows && !own_grouping_pays(bytes, own_sizes, sizes)) {
      rows.own_rows = false;
      for (size_t i = 0; i < n; ++i)
        if (place[i].kind == eco::UNIT_WIDE)
          place[i] = eco::place_tensor(tensors[i].numel, place[i].group, eco::GROUP_WIDE, true, tensors[i].fmt, eco::TILE_ELEMS, 0, &rows);
    }
    e = hipGetDevice(&plan->device);
    if (e != hipSuccess) { delete plan; return fail_hip(e, "hipGetDevice"); }
    plan->cus = num_compute_units();
    const int plain_home = home_of_plain(tensors_of, entries_of);
    const auto home = [&](size_t i) {
      const int f = tensors[i].fmt;
      return f == ECO_FMT_FP8_E4M3 || f == ECO_FMT_INT4 || plain_home < 0 ? f : plain_home;
    };
    // tensors with one scale that the chip can hold: one pass, if it pays for those of the format
    const uint64_t max_slabs = std::min<uint64_t>(eco::RES_WAVES * 64, eco::RES_SLABS_PER_WG * plan->cus);
    for (int f = 0; f < 2; ++f) {
      uint64_t bytes = 0, slabs = 0;
      uint64_t odd = 0;
      bool any = false, tails = false, longer = false, listed = false;
      const auto in_one_pass = [&](size_t i) {
        return eco::place_tensor(tensors[i].numel, tensors[i].numel, eco::GROUP_TENSOR, true, tensors[i].fmt, eco::RES_SLAB, max_slabs);
      };
      const auto count = [&](size_t i) {
        const eco::Placement p = in_one_pass(i);
        any = true;
        if (p.list != eco::LIST_RESIDENT) { longer = true; return; }
        bytes += eco::array_bytes(tensors[i].numel, f, state);
        slabs += p.units;
        tails = tails || tensors[i].numel % eco::ELEMS_PER_LANE != 0;
      };
      for (size_t i = 0; i < n; ++i) {
        if (home(i) != f) continue;
        if (place[i].list == eco::LIST_TW_TILES) count(i);
        else if (short_odd(tensors[i], layout)) odd += place[i].entries;
        else listed = true;
      }
      const unsigned cus = static_cast<unsigned>(plan->cus);
      if (any && odd && odd <= ODD_ALONG_ENTRIES &&
          (tails || !eco::one_pass_pays(state, bytes, slabs, cus, tails, longer) || (!listed && slabs <= cus)))
        for (size_t i = 0; i < n; ++i)
          if (tensors[i].fmt == f && short_odd(tensors[i], layout)) {
            place[i] = eco::place_tensor(tensors[i].numel, tensors[i].numel, eco::GROUP_TENSOR, true, f);
            count(i);
          }
      if (!eco::one_pass_pays(state, bytes, slabs, cus, tails, longer)) continue;
      for (size_t i = 0; i < n; ++i)
        if (tensors[i].fmt == f && place[i].list == eco::LIST_TW_TILES) place[i] = in_one_pass(i);
    }

    uint64_t elements[4] = {0};
    descs.reserve(n);
    for (size_t i = 0; i < n; ++i) {
      const eco_tensor_t &t = tensors[i];
      const eco::Placement &p = place[i];
      const int f = home(i);
      Lists &g = plan->lists[f];
      const uint32_t idx = static_cast<uint32_t>(i);
      std::vector<uint32_t> &list = g.list(p.list);
      eco::TensorDesc d = describe(t, layout, p, list.size());
      if (p.list == eco::LIST_TW_TILES || p.list == eco::LIST_RESIDENT) {
        g.load[eco::STREAM_TENSORWISE].elements += t.numel;
        g.load[eco::STREAM_TENSORWISE].off_lines += off_lines(t, p, state) ? t.numel : 0;
      }
      if (p.list == eco::LIST_TW_TILES) {
        d.slot = static_cast<uint32_t>(g.tw_tensor.size());
        g.tw_tensor.push_back(idx);
        g.most_tw_tiles = std::max(g.most_tw_tiles, p.units);
      } else if (p.list == eco::LIST_RESIDENT) {
        d.slot = static_cast<uint32_t>(t.numel % eco::ELEMS_PER_LANE);
        d.numel = t.numel - d.slot;
        d.group_size = g.resident.size();             // its place in the list
        g.tails += d.slot != 0;
        g.resident.push_back(idx);
      } else {
        elements[f] += t.numel;
        Lists::WideLoad &w = g.load[p.kind == eco::UNIT_WIDE ? p.list - eco::LIST_WIDE1 + 1 : 0];
        if (p.kind == eco::UNIT_WIDE) w.idle += p.idle ? p.units : 0;
        if (p.list != eco::LIST_TILE) w.elements += t.numel;
        if (off_lines(t, p, state)) w.off_lines += t.numel;
      }
      list.insert(list.end(), static_cast<size_t>(p.units), idx);
      if (p.tail) {
        g.extra.push_back(idx);
        g.load[0].elements += t.numel % eco::TILE_ELEMS;
      }
      g.tensors += 1;
      descs.push_back(d);
    }
    for (int f = 0; f < 2; ++f) {
      Lists &g = plan->lists[f];
      int launches = g.tile.empty() ? 0 : 1;
      for (int nw = 1; nw <= eco::MAX_WIDE_WAVES; ++nw) launches += !g.wide[nw].empty();
      if (launches < 2 || elements[f] > SMALL_ELEMENTS) continue;
      const auto listed = [&](size_t i) { return home(i) == f && place[i].list != eco::LIST_TW_TILES && place[i].list != eco::LIST_RESIDENT; };
      for (size_t i = 0; i < n; ++i)
        if (listed(i)) g.one_waves = std::max(g.one_waves, unit_waves(place[i]));
      for (size_t i = 0; i < n; ++i) {
        if (!listed(i)) continue;
        const uint32_t idx = static_cast<uint32_t>(descs.size());
        descs.push_back(describe_in_list(tensors[i], layout, place[i], g.one.size()));
        g.one.insert(g.one.end(), static_cast<size_t>(list_workgroups(place[i], g.one_waves)), idx);
      }
    }

    // one device buffer: per format [full tiles | one-wave units (right behind: see eco_step_kernel) | all of a list launch | wide lists 1..16 | tensor-wise tiles | tensor-wise tensors | slots |
    // tile maxima | slabs | their tensors | tail maxima | slab maxima | counts | deferred slabs]
    for (Lists &g : plan->lists) {
      const auto add = [&host](const std::vector<uint32_t> &l, size_t *off) {
        *off = host.size();
        host.insert(host.end(), l.begin(), l.end());
      };
      if (!g.tensors) continue;
      add(g.tile, &g.off_tile);
      add(g.extra, &g.off_extra);
      add(g.one, &g.off_one);
      for (int nw = 1; nw <= eco::MAX_WIDE_WAVES; ++nw) add(g.wide[nw], &g.off_wide[nw]);
      add(g.tw_tile, &g.off_tw_tile);
      add(g.tw_tensor, &g.off_tw_tensor);
      g.off_slots = host.size();
      host.insert(host.end(), g.tw_tensor.size() + 1, 0u);      // abs-max slots start at zero
      g.off_tile_max = host.size();
      host.insert(host.end(), g.tw_tile.size(), 0u);
      add(g.slab, &g.off_slab);
      add(g.resident, &g.off_resident);
      g.off_tail_max = host.size();
      host.insert(host.end(), g.resident.size(), 0u);
      g.off_slab_max = host.size();
      host.insert(host.end(), g.slab.size(), 0xFFFFFFFFu);      // no slab's maximum is known
      g.off_counts = host.size();
      host.insert(host.end(), 2, 0u);
      g.off_deferred = host.size();
      host.insert(host.end(), g.slab.size(), 0u);
    }
  } catch (const std::bad_alloc &) {
    delete plan;
    return fail(ECO_ENOMEM, "plan: host allocation failed");
  }

  e = hipMalloc(reinterpret_cast<void **>(&plan->d_descs), descs.size() * sizeof(eco::TensorDesc));
  if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void **>(&plan->d_tables), host.size() * sizeof(uint32_t));
  if (e == hipSuccess) e = hipMemcpy(plan->d_descs, descs.data(), descs.size() * sizeof(eco::TensorDesc), hipMemcpyHostToDevice);
  if (e == hipSuccess) e = hipMemcpy(plan->d_tables, host.data(), host.size() * sizeof(uint32_t), hipMemcpyHostToDevice);
  if (e != hipSuccess) {
    st = (e == hipErrorOutOfMemory) ? fail(ECO_ENOMEM, "plan: device allocation failed") : fail_hip(e, "plan upload");
    (void)eco_plan_destroy(plan);
    return st;
  }
  for (int f = 0; f < 4; ++f) {
    Lists &g = plan->lists[f];
    if (!g.tensors) continue;
    eco::StepLaunch &sl = g.launch;
    eco::StepArgs &a = sl.args;
    a.tensors = plan->d_descs;
    sl.tile_tensor = plan->d_tables + g.off_tile;
    a.extra_tensor = plan->d_tables + g.off_extra;
    a.num_tiles = static_cast<uint32_t>(g.tile.size());
    a.num_extra = static_cast<uint32_t>(g.extra.size());
    sl.wide_base = plan->d_tables;
    for (int nw = 1; nw <= eco::MAX_WIDE_WAVES; ++nw) {
      sl.wide_offset[nw] = static_cast<uint32_t>(g.off_wide[nw]);
      sl.num_wide[nw] = static_cast<uint32_t>(g.wide[nw].size());
    }
    a.tw_tile_tensor = plan->d_tables + g.off_tw_tile;
    a.tw_tensor = plan->d_tables + g.off_tw_tensor;
    a.slots = plan->d_tables + g.off_slots;
    a.tile_max = plan->d_tables + g.off_tile_max;
    a.num_tw_tiles = static_cast<uint32_t>(g.tw_tile.size());
    a.num_tw_tensors = static_cast<uint32_t>(g.tw_tensor.size());
    a.tw_reduce_wgs = eco::tw_reduce_workgroups(g.most_tw_tiles);
    a.slab_tensor = plan->d_tables + g.off_slab;
    a.slab_max = plan->d_tables + g.off_slab_max;
    a.resident_counts = plan->d_tables + g.off_counts;
    a.deferred = plan->d_tables + g.off_deferred;
    a.resident_tensor = plan->d_tables + g.off_resident;
    a.num_resident = static_cast<uint32_t>(g.resident.size());
    a.resident_tails = static_cast<uint32_t>(g.tails);
    a.tail_max = plan->d_tables + g.off_tail_max;
    a.num_slabs = static_cast<uint32_t>(g.slab.size());
    a.resident_tries = eco::RES_TRIES;
    sl.resident_wgs = static_cast<unsigned>(plan->cus);
    sl.list_tensor = plan->d_tables + g.off_one;
    sl.list_wgs = g.one.size();
    sl.list_waves = g.one_waves;
    choose_launches(variant_for(layout, f), g.load, bytes, &sl);
  }
  *out = plan;
  return ECO_OK;
}

// Launches the step of one format's lists (sl: everything but the scalars).
static eco_status_t launch_format(const eco_hparams_t *hp, const eco_constants_t &c, const eco::KernelVariant &kv, int cus, eco::StepLaunch *sl,
                                  eco::SmallArgs *small, hipStream_t stream) {
  fill_step_scalars(hp, c, sl);
  sl->max_tile_threads = tile_threads(sl->max_launch_threads, cus);
  if (small) {
    sl->args.wg_waves = sl->list_waves;
    small->step = sl->args;
    sl->small = small;
  }
  const hipError_t e = eco::launch_step(kv, *sl, stream);
  return e == hipSuccess ? ECO_OK : fail_hip(e, "step kernel launch");
}

eco_status_t eco_step(eco_plan_t *plan, const eco_hparams_t *hp, void *stream) {
  if (!plan) return fail(ECO_EINVAL, "step: null plan");
  eco_status_t st = check_hparams(hp);
  if (st != ECO_OK) return st;
  if (hp->block_size != plan->block_size || hp->state_dtype != plan->state_dtype || hp->scale_dtype != plan->scale_dtype ||
      hp->opt != plan->opt || hp->mode != plan->mode)
    return fail(ECO_EINVAL, "step: block_size, state_dtype, scale_dtype, opt and mode must equal the plan's");
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess || dev != plan->device)
    return fail(ECO_EINVAL, "step: the plan was created on device %d, which is not the current device (%d)", plan->device, dev);
  (void)hipGetLastError();   // an error left behind by the caller's earlier HIP work is not this call's

  if (!plan->d_descs || !plan->d_tables) return fail(ECO_EINVAL, "step: the plan's device tables are missing");
  eco_constants_t c;
  derive_constants(hp, &c);
  if (plan->unfinished) {
    const hipError_t e = reset_scratch(*plan, static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return fail_hip(e, "scratch kernel launch");
  }
  plan->unfinished = true;
  for (int f = 0; f < 4; ++f) {
    const Lists &g = plan->lists[f];
    if (!g.tensors) continue;
    eco::StepLaunch sl = g.launch;
    st = launch_format(hp, c, variant_for(hp, f), plan->cus, &sl, nullptr, static_cast<hipStream_t>(stream));
    if (st != ECO_OK) return st;
  }
  plan->unfinished = false;
  return ECO_OK;
}

eco_status_t eco_step_tensors(const eco_tensor_t *tensors, size_t n, const eco_hparams_t *hp, void *stream) {
  eco_status_t st = check_hparams(hp);
  if (st != ECO_OK) return st;
  eco_plan_t *plan = nullptr;
  st = eco_plan_create(tensors, n, hp, &plan);
  if (st != ECO_OK) return st;
  st = eco_step(plan, hp, stream);
  const hipError_t e = hipStreamSynchronize(static_cast<hipStream_t>(stream));
  const eco_status_t st2 = eco_plan_destroy(plan);
  if (st != ECO_OK) return st;
  if (e != hipSuccess) return fail_hip(e, "hipStreamSynchronize");
  return st2;
}

eco_status_t eco_step_tensors_noalloc(const eco_tensor_t *tensors, size_t n, const eco_hparams_t *hp, void *stream) {
  using namespace noalloc;
  eco_status_t st = check_hparams(hp);
  if (st != ECO_OK) return st;
  st = check_layout(hp);
  if (st != ECO_OK) return st;
  if (!tensors || n == 0) return fail(ECO_EINVAL, "step: empty tensor list");
  if (n > MAX_TENSORS)
    return fail(ECO_EUNSUPPORTED, "eco_step_tensors_noalloc: %zu tensors, the static scratch holds %u (use a plan)", n, MAX_TENSORS);

  // pass 1: validate, place, count the entries of every launch list
  constexpr int L_TW_TENSORS = eco::LIST_COUNT, L_COUNT = eco::LIST_COUNT + 1;
  uint64_t count[4][L_COUNT] = {{0}}, tensors_of[4] = {0}, entries_of[4] = {0}, most_tw_tiles[4] = {0};
  uint64_t total = 0, elements = 0, bytes = 0;
  const eco::StateLayout state = state_layout(hp);
  WideLoads load[4] = {};
  // The placement of a tensor that check_tensor has let through: rows first as the limit on launch tables counts them.
  eco::StepRows rows = {state, false};
  bool odd_along[2] = {false, false};      // see short_odd: along with the longer ones of the format
  const auto place = [&](const eco_tensor_t &t) {
    const bool quantized = t.fmt == ECO_FMT_FP8_E4M3 || t.fmt == ECO_FMT_INT4;
    const uint64_t gsz = t.group_size ? t.group_size : hp->block_size;
    const int cls = quantized ? eco::classify_group(gsz, t.numel) : eco::GROUP_BLOCK;
    return eco::place_tensor(t.numel, gsz, cls, quantized, t.fmt, eco::TILE_ELEMS, 0, cls == eco::GROUP_TENSOR && odd_along[t.fmt] ? nullptr : &rows);
  };
  uint64_t units = 0;
  const auto count_wide = [&](const eco_tensor_t &t, const eco::Placement &p) {
    Lists::WideLoad &w = load[t.fmt][p.list - eco::LIST_WIDE1 + 1];
    count[t.fmt][p.list] += p.units;
    units += p.units;
    w.idle += p.idle ? p.units : 0;
    w.elements += t.numel;
  };
  const auto count_tensorwise = [&](int f, const eco_tensor_t &t, const eco::Placement &p) {
    count[f][eco::LIST_TW_TILES] += p.units;
    count[f][L_TW_TENSORS] += 1;
    load[f][eco::STREAM_TENSORWISE].elements += t.numel;
    units += p.units + 1;
    most_tw_tiles[f] = std::max(most_tw_tiles[f], p.units);
  };
  bool tensorwise = false, wide = false;
  uint64_t odd_entries[4] = {0};
  for (size_t i = 0; i < n; ++i) {
    const int f = tensors[i].fmt;
    uint64_t gsz = 0;
    int cls = 0;
    st = check_tensor(tensors[i], i, hp, &gsz, &cls);
    if (st != ECO_OK) return st;
    const eco::Placement p = place(tensors[i]);
    if (p.entries > MAX_UNITS) return fail(ECO_EUNSUPPORTED, "eco_step_tensors_noalloc: tensor %zu alone exceeds the static scratch", i);
    tensors_of[f] += 1;
    entries_of[f] += p.entries;
    elements += tensors[i].numel;
    bytes += eco::array_bytes(tensors[i].numel, f, state);
    total += p.entries;
    if (total > MAX_UNITS)
      return fail(ECO_EUNSUPPORTED, "eco_step_tensors_noalloc: more than %u launch-table entries (512-element tiles, or scale "
                  "groups wider than 512): the static scratch does not hold them (use a plan)", MAX_UNITS);
    if (p.list == eco::LIST_TW_TILES) {
      tensorwise = true;
      count_tensorwise(f, tensors[i], p);
      continue;
    }
    if (cls == eco::GROUP_TENSOR) odd_entries[f] += p.entries;
    if (p.kind == eco::UNIT_WIDE) {
      wide = true;
      count_wide(tensors[i], p);
      continue;
    }
    count[f][p.list] += p.units;
    units += p.units;
    if (p.list == eco::LIST_EXTRA) load[f][0].elements += tensors[i].numel;
    if (p.tail) {
      count[f][eco::LIST_EXTRA] += 1;
      units += 1;
      load[f][0].elements += tensors[i].numel % eco::TILE_ELEMS;
    }
  }
  const int plain_home = home_of_plain(tensors_of, entries_of);
  for (int f = 0; f < 2; ++f) {
    if (!odd_entries[f] || odd_entries[f] > ODD_ALONG_ENTRIES || !count[f][L_TW_TENSORS]) continue;
    for (size_t i = 0; i < n; ++i) {
      if (tensors[i].fmt != f || !short_odd(tensors[i], hp)) continue;
      const eco::Placement p = place(tensors[i]);
      count[f][p.list] -= p.units;
      units -= p.units;
      Lists::WideLoad &w = load[f][p.kind == eco::UNIT_WIDE ? p.list - eco::LIST_WIDE1 + 1 : 0];
      w.idle -= p.idle ? p.units : 0;
      w.elements -= tensors[i].numel;
    }
    odd_along[f] = true;
    for (size_t i = 0; i < n; ++i)
      if (tensors[i].fmt == f && short_odd(tensors[i], hp)) count_tensorwise(f, tensors[i], place(tensors[i]));
  }
  // The wide lists again with the step's own grouping of rows, where it is the better one (see bytes_of, own_grouping_pays) and the
  // static tables hold its units; back to the other one if not.
  const bool own = wide && HbmBound(bytes).half;
  uint32_t sizes[2][4] = {{0}};
  const auto used = [&](uint32_t (&bits)[4]) {
    for (int f = 0; f < 4; ++f)
      for (int nw = 1; nw <= eco::MAX_WIDE_WAVES; ++nw) bits[f] |= (count[f][eco::LIST_WIDE1 + nw - 1] ? 1u : 0u) << (nw - 1);
  };
  if (own) used(sizes[0]);
  for (int round = 0; own && round < 2; ++round) {
    rows.own_rows = round == 0;
    for (int f = 0; f < 4; ++f)
      for (int nw = 1; nw <= eco::MAX_WIDE_WAVES; ++nw) {
        units -= count[f][eco::LIST_WIDE1 + nw - 1];
        count[f][eco::LIST_WIDE1 + nw - 1] = 0;
        load[f][nw] = Lists::WideLoad{0, 0, 0};
      }
    for (size_t i = 0; i < n; ++i) {
      const eco::Placement p = place(tensors[i]);
      if (p.kind == eco::UNIT_WIDE) count_wide(tensors[i], p);
    }
    if (round == 0) used(sizes[1]);
    if (units <= MAX_UNITS && own_grouping_pays(bytes, sizes[1], sizes[0])) break;
  }
  const auto format_of = [&](size_t i) {
    const int32_t fmt = tensors[i].fmt;
    return fmt == ECO_FMT_FP8_E4M3 || fmt == ECO_FMT_INT4 || plain_home < 0 ? fmt : plain_home;
  };
  for (int f = eco::FMT_BF16_PLAIN; f <= eco::FMT_FP32_ID && plain_home >= 0; ++f) {
    count[plain_home][eco::LIST_EXTRA] += count[f][eco::LIST_EXTRA];
    load[plain_home][0].elements += load[f][0].elements;
    count[f][eco::LIST_EXTRA] = 0;
  }
  if (bytes >= stream_from(!state.state_bf16))
    for (size_t i = 0; i < n; ++i) {
      const eco::Placement p = place(tensors[i]);
      const int l = p.list == eco::LIST_TW_TILES ? eco::STREAM_TENSORWISE : p.kind == eco::UNIT_WIDE ? p.list - eco::LIST_WIDE1 + 1 : 0;
      if (off_lines(tensors[i], p, state)) load[format_of(i)][l].off_lines += tensors[i].numel;
    }
  (void)hipGetLastError();
  hipStream_t hs = static_cast<hipStream_t>(stream);
  eco_constants_t c;
  derive_constants(hp, &c);
  const int cus = num_compute_units();

  // lists of small tensors need no tables: their descriptors go as kernel arguments, SMALL_TENSORS to a launch (205 tensors, us: with
  // tables, which take seven launches to write, 35.6; in five launches 23.6)
  if (!tensorwise && elements <= SMALL_ELEMENTS && (plain_home >= 0 || !(tensors_of[2] + tensors_of[3])) && tensors_of[0] + tensors_of[1]) {
    SmallItem items[eco::SMALL_TENSORS];                // no container: this call allocates nothing, on the host neither
    eco::SmallArgs small;
    eco::StepLaunch sl;
    const int64_t limit = g_max_launch_threads.load(std::memory_order_relaxed);
    // (a limit on a launch's threads holds here too: a first round without launching, if there is one)
    bool fits = true;
    for (int round = limit > 0 ? 0 : 1; round < 2 && fits; ++round)
      for (int f = 0; f < 2; ++f) {
        size_t held = 0;
        for (size_t i = 0; i <= n && fits; ++i) {
          if (i < n && format_of(i) == f) {
            ::new (&items[held++]) SmallItem{&tensors[i], place(tensors[i])};      // (built where it lies: a copy is 5 ns)
          }
          if (!held || (held < static_cast<size_t>(eco::SMALL_TENSORS) && i < n)) continue;
          std::memset(&sl, 0, sizeof sl);
          make_small(items, held, hp, &small, &sl.list_wgs, &sl.list_waves);
          held = 0;
          if (round == 0) { fits = sl.list_wgs * sl.list_waves * 64 <= static_cast<uint64_t>(limit); continue; }
          st = launch_format(hp, c, variant_for(hp, f), cus, &sl, &small, hs);
          if (st != ECO_OK) return st;
        }
      }
    if (fits) return ECO_OK;
  }

  uint32_t start[4][L_COUNT], tw_tile_start[4], tw_tensor_start[4];
  {
    uint32_t pos = 0, tw_tiles = 0, tw_tensors = 0;
    for (int f = 0; f < 4; ++f) {
      for (int l = 0; l < L_COUNT; ++l) { start[f][l] = pos; pos += static_cast<uint32_t>(count[f][l]); }
      tw_tile_start[f] = tw_tiles; tw_tiles += static_cast<uint32_t>(count[f][eco::LIST_TW_TILES]);
      tw_tensor_start[f] = tw_tensors; tw_tensors += static_cast<uint32_t>(count[f][L_TW_TENSORS]);
    }
  }

  unsigned char *sp = nullptr;
  st = scratch_for_current_device(&sp);
  if (st != ECO_OK) return st;

  // pass 2: descriptors and tables, BUILD_CHUNK tensors per launch of the builder
  uint32_t fill[4][L_COUNT] = {{0}};
  BuildArgs ba;
  std::memset(&ba, 0, sizeof ba);
  ba.scratch = sp;
  for (size_t i = 0; i < n; ++i) {
    const eco::Placement p = place(tensors[i]);
    const int f = format_of(i);
    const uint32_t k = ba.count++;
    if (k == 0) ba.first_index = static_cast<uint32_t>(i);
    eco::TensorDesc &d = ba.desc[k];
    d = describe(tensors[i], hp, p, fill[f][p.list]);
    ba.list_pos[k] = start[f][p.list] + fill[f][p.list];
    ba.units[k] = static_cast<uint32_t>(p.units);
    fill[f][p.list] += static_cast<uint32_t>(p.units);
    ba.extra_pos[k] = ba.slot_pos[k] = NO_ENTRY;
    if (p.tail) ba.extra_pos[k] = start[f][eco::LIST_EXTRA] + fill[f][eco::LIST_EXTRA]++;
    if (p.list == eco::LIST_TW_TILES) {
      d.slot = fill[f][L_TW_TENSORS];
      ba.slot_pos[k] = tw_tensor_start[f] + d.slot;
      ba.extra_pos[k] = start[f][L_TW_TENSORS] + fill[f][L_TW_TENSORS]++;
    }
    if (ba.count == BUILD_CHUNK || i + 1 == n) {
      hipLaunchKernelGGL(eco_noalloc_build_kernel, dim3(ba.count, BUILD_BLOCKS_PER_TENSOR), dim3(BUILD_THREADS), 0, hs, ba);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return fail_hip(e, "table kernel launch");
      ba.count = 0;
    }
  }

  const eco::TensorDesc *descs = reinterpret_cast<const eco::TensorDesc *>(sp + OFF_DESCS);
  uint32_t *tables = reinterpret_cast<uint32_t *>(sp + OFF_TABLES);
  for (int f = 0; f < 4; ++f) {
    uint64_t any = 0;
    for (int l = 0; l < L_COUNT; ++l) any += count[f][l];
    if (!any) continue;
    eco::StepLaunch sl;
    std::memset(&sl, 0, sizeof sl);
    eco::StepArgs &a = sl.args;
    a.tensors = descs;
    sl.tile_tensor = tables + start[f][eco::LIST_TILE];
    a.extra_tensor = tables + start[f][eco::LIST_EXTRA];
    a.num_tiles = static_cast<uint32_t>(count[f][eco::LIST_TILE]);
    a.num_extra = static_cast<uint32_t>(count[f][eco::LIST_EXTRA]);
    sl.wide_base = tables;
    for (int nw = 1; nw <= eco::MAX_WIDE_WAVES; ++nw) {
      sl.wide_offset[nw] = start[f][eco::LIST_WIDE1 + nw - 1];
      sl.num_wide[nw] = static_cast<uint32_t>(count[f][eco::LIST_WIDE1 + nw - 1]);
    }
    a.tw_tile_tensor = tables + start[f][eco::LIST_TW_TILES];
    a.tw_tensor = tables + start[f][L_TW_TENSORS];
    a.slots = reinterpret_cast<uint32_t *>(sp + OFF_SLOTS) + tw_tensor_start[f];
    a.tile_max = reinterpret_cast<uint32_t *>(sp + OFF_TILE_MAX) + tw_tile_start[f];
    a.num_tw_tiles = static_cast<uint32_t>(count[f][eco::LIST_TW_TILES]);
    a.num_tw_tensors = static_cast<uint32_t>(count[f][L_TW_TENSORS]);
    a.tw_reduce_wgs = eco::tw_reduce_workgroups(most_tw_tiles[f]);
    const eco::KernelVariant kv = variant_for(hp, f);
    choose_launches(kv, load[f], bytes, &sl);
    st = launch_format(hp, c, kv, cus, &sl, nullptr, hs);
    if (st != ECO_OK) return st;
  }
  return ECO_OK;
}

static eco_status_t check_flat(const void *weights, const void *scales, uint64_t numel, int32_t fmt, uint64_t group_size,
                               int32_t scale_dtype) {
  if (fmt != ECO_FMT_FP8_E4M3 && fmt != ECO_FMT_INT4) return fail(ECO_EINVAL, "format %d is not a quantized format", fmt);
  if (!is_dtype(scale_dtype)) return fail(ECO_EINVAL, "unknown scale dtype");
  if (numel == 0) return fail(ECO_EINVAL, "numel == 0");
  if (numel > (1ull << 40)) return fail(ECO_EUNSUPPORTED, "more than 2^40 elements in one call");
  if (group_size == 0) return fail(ECO_EINVAL, "group_size must be positive");
  if (!weights || !scales) return fail(ECO_EINVAL, "null weights or scales");
  if (!aligned16(weights) || !aligned16(scales)) return fail(ECO_EALIGN, "weights and scales must be 16-byte aligned");
  if (!eco::flat_call_fits(numel, group_size))
    return fail(ECO_EUNSUPPORTED, "%llu elements in groups of %llu: one call handles what one launch can (about 2^35 elements); "
                "call it on slices of whole scale groups", (unsigned long long)numel, (unsigned long long)group_size);
  return ECO_OK;
}

eco_status_t eco_quantize_init(const void *src, int32_t src_dtype, uint64_t numel, int32_t fmt, uint64_t group_size,
                               int32_t scale_dtype, void *weights, void *scales, void *stream) {
  eco_status_t st = check_flat(weights, scales, numel, fmt, group_size, scale_dtype);
  if (st != ECO_OK) return st;
  if (!src) return fail(ECO_EINVAL, "null source");
  if (!is_dtype(src_dtype)) return fail(ECO_EINVAL, "unknown source dtype");
  if (!aligned16(src)) return fail(ECO_EALIGN, "source must be 16-byte aligned");
  if (eco::classify_group(group_size, numel) == eco::GROUP_UNSUPPORTED)
    return fail(ECO_EUNSUPPORTED, "scale group of %llu elements: supported are powers of two in [32, 512], multiples of 8 "
                "up to 8192, and the whole tensor", (unsigned long long)group_size);
  (void)hipGetLastError();
  const hipError_t e = eco::launch_quantize_init(src, src_dtype == ECO_DT_BF16, numel, fmt, group_size,
                                                 scale_dtype == ECO_DT_BF16, weights, scales, static_cast<hipStream_t>(stream));
  return e == hipSuccess ? ECO_OK : fail_hip(e, "quantize kernel launch");
}

eco_status_t eco_dequantize(const void *weights, const void *scales, uint64_t numel, int32_t fmt, uint64_t group_size,
                            int32_t scale_dtype, float *dst, void *stream) {
  eco_status_t st = check_flat(weights, scales, numel, fmt, group_size, scale_dtype);
  if (st != ECO_OK) return st;
  if (!dst) return fail(ECO_EINVAL, "null destination");
  if (!aligned16(dst)) return fail(ECO_EALIGN, "destination must be 16-byte aligned");
  if (group_size < 8 && group_size < numel)      // a single group over a tiny tensor is fine
    return fail(ECO_EUNSUPPORTED, "scale groups of fewer than 8 elements are not supported");
  (void)hipGetLastError();
  const hipError_t e = eco::launch_dequantize(weights, scales, numel, fmt, group_size, scale_dtype == ECO_DT_BF16, nullptr, 0,
                                              dst, static_cast<hipStream_t>(stream));
  return e == hipSuccess ? ECO_OK : fail_hip(e, "dequantize kernel launch");
}

eco_status_t eco_quantize_error(const void *src, int32_t src_dtype, const void *weights, const void *scales, uint64_t numel,
                                int32_t fmt, uint64_t group_size, int32_t scale_dtype, float *err, void *stream) {
  eco_status_t st = check_flat(weights, scales, numel, fmt, group_size, scale_dtype);
  if (st != ECO_OK) return st;
  if (!src || !err) return fail(ECO_EINVAL, "null source or destination");
  if (!is_dtype(src_dtype)) return fail(ECO_EINVAL, "unknown source dtype");
  if (!aligned16(src) || !aligned16(err)) return fail(ECO_EALIGN, "source and destination must be 16-byte aligned");
  if (group_size < 8 && group_size < numel)
    return fail(ECO_EUNSUPPORTED, "scale groups of fewer than 8 elements are not supported");
  (void)hipGetLastError();
  const hipError_t e = eco::launch_dequantize(weights, scales, numel, fmt, group_size, scale_dtype == ECO_DT_BF16, src,
                                              src_dtype == ECO_DT_BF16 ? 2 : 1, err, static_cast<hipStream_t>(stream));
  return e == hipSuccess ? ECO_OK : fail_hip(e, "quantization-error kernel launch");
}

eco_status_t eco_bandwidth_probe(int32_t kind, void *codes, void *scales, const void *grad, void *m, void *v, uint64_t numel,
                                 void *stream) {
  if (kind != 0 && kind != 1) return fail(ECO_EINVAL, "probe kind %d: 0 = byte-mix copy, 1 = plain copy", kind);
  if (!m || !v || (kind == 0 && (!codes || !scales || !grad))) return fail(ECO_EINVAL, "null array");
  if (!aligned16(m) || !aligned16(v) || (kind == 0 && (!aligned16(codes) || !aligned16(scales) || !aligned16(grad))))
    return fail(ECO_EALIGN, "every array must be 16-byte aligned");
  if (numel == 0 || numel % 1024 != 0 || numel / eco::ELEMS_PER_LANE > eco::MAX_LAUNCH_THREADS)
    return fail(ECO_EINVAL, "numel must be a positive multiple of 1024 below 2^35");
  eco::KernelVariant kv;
  kv.fmt = eco::FMT_FP8; kv.state_bf16 = 0; kv.scale_bf16 = 0; kv.algo = eco::ALGO_ADAM; kv.round = eco::ROUND_SR;
  const uint64_t bytes = numel * (kind == 0 ? 11 : 8);
  const bool streamed = bytes >= stream_from(true);
  const int64_t opt_lds = g_lds_bytes.load(std::memory_order_relaxed);
  const uint32_t lds = opt_lds >= 0 ? static_cast<uint32_t>(opt_lds)
                                    : lds_for_waves(streamed ? streaming_waves(kv, bytes) : default_waves(kv, HbmBound(bytes)), 512);
  (void)hipGetLastError();
  const hipError_t e = eco::launch_bandwidth_probe(kind, codes, scales, grad, m, v, numel, streamed, lds, static_cast<hipStream_t>(stream));
  return e == hipSuccess ? ECO_OK : fail_hip(e, "probe kernel launch");
}

eco_status_t eco_arith_selftest(int32_t kind, float numerator, uint32_t bits_lo, uint32_t bits_hi, uint64_t *mismatches,
                                void *stream) {
  if (kind != 0 && kind != 1) return fail(ECO_EINVAL, "self-test kind %d: 0 = square root, 1 = division", kind);
  if (!mismatches || (reinterpret_cast<uintptr_t>(mismatches) & 7u)) return fail(ECO_EINVAL, "mismatch counter: null or not 8-byte aligned");
  if (bits_hi <= bits_lo) return fail(ECO_EINVAL, "empty range of bit patterns");
  // the ranges the short forms are used in (bit patterns of positive floats)
  const uint32_t lo = kind == 0 ? 0x0F800000u : 0x27800000u, hi = kind == 0 ? 0x6F800001u : 0x58000001u;   // 2^-96..2^96 | 2^-48..2^49
  if (bits_lo < lo || bits_hi > hi) return fail(ECO_EINVAL, "bit patterns outside the range the short form is used in");
  if (kind == 1 && !(std::fabs(numerator) >= 0x1p-40f && std::fabs(numerator) <= 0x1p40f))
    return fail(ECO_EINVAL, "numerator outside [2^-40, 2^40]");
  (void)hipGetLastError();
  const hipError_t e = eco::launch_arith_selftest(kind, numerator, bits_lo, bits_hi, reinterpret_cast<unsigned long long *>(mismatches),
                                                  static_cast<hipStream_t>(stream));
  return e == hipSuccess ? ECO_OK : fail_hip(e, "self-test kernel launch");
}

eco_status_t eco_philox_fill(uint64_t seed, uint64_t step, uint32_t tensor_id, uint64_t first_word, uint64_t n_words,
                             uint32_t *dst, void *stream) {
  if (!dst) return fail(ECO_EINVAL, "null destination");
  if (n_words == 0) return fail(ECO_EINVAL, "n_words == 0");
  if (first_word + n_words < first_word) return fail(ECO_EINVAL, "word range overflows");
  (void)hipGetLastError();
  const hipError_t e = eco::launch_philox_fill(seed, step, tensor_id, first_word, n_words, dst, static_cast<hipStream_t>(stream));
  return e == hipSuccess ? ECO_OK : fail_hip(e, "philox kernel launch");
}

}  // extern "C"
