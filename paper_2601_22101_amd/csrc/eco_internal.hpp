// Host/device shared declarations of the ECO library: launch tables and launcher entry points.
#pragma once
#include <hip/hip_runtime_api.h>
#include <stdint.h>

namespace eco {

enum : int { FMT_FP8 = 0, FMT_INT4 = 1, FMT_BF16_PLAIN = 2, FMT_FP32_ID = 3 };
enum : int { ROUND_SR = 0, ROUND_RTN = 1 };
// optimizer x treatment of the quantization error: Adam / SGDM with the memory-free injection (or none,
// when the injection constants are zero), SGDM with the exact stored-error injection, and the
// master-weight baselines
enum : int { ALGO_ADAM = 0, ALGO_SGDM = 1, ALGO_SGDM_EXACT = 2, ALGO_ADAM_MASTER = 3, ALGO_SGDM_MASTER = 4 };
constexpr bool algo_is_adam(int a) { return a == ALGO_ADAM || a == ALGO_ADAM_MASTER; }
constexpr bool algo_is_master(int a) { return a == ALGO_ADAM_MASTER || a == ALGO_SGDM_MASTER; }

// A tile is TILE_ELEMS consecutive elements of one tensor, processed by one workgroup of one wave,
// 8 consecutive elements per lane.  A scale group of B elements therefore occupies B/8 consecutive
// lanes (B = 32..512 fits inside the 64-lane wave).
#ifndef ECO_WG_THREADS
#define ECO_WG_THREADS 64
#endif
constexpr int WG_THREADS = ECO_WG_THREADS;
constexpr int ELEMS_PER_LANE = 8;
constexpr int TILE_ELEMS = WG_THREADS * ELEMS_PER_LANE;

// Limits of the allocation-free plan-less step (its tables live in a static device array): tensors per call,
// and launch-table entries per call (one per 512-element tile; one per scale group for groups wider than that).
#define ECO_NOALLOC_MAX_TENSORS 4096
#define ECO_NOALLOC_MAX_UNITS (1u << 20)

constexpr int MAX_WIDE_WAVES = 16;          // widest single-workgroup scale group: 16 waves * 512 = 8192 elements
constexpr uint64_t MAX_WIDE_GROUP = 8192;

// What a wave does with one of its tensor's units.  Full 512-element tiles of block-scaled tensors and groups of more
// than 512 elements have launch lists of their own; everything else a step consists of -- the last, partial tile of a
// block-scaled tensor, groups of up to 512 elements that are no power of two, unquantized tensors -- is a list of
// one-wave units that ride in the launch of those (StepArgs::extra_tensor).
enum : int {
  UNIT_TILES = 0,       // block-scaled: unit u is tile u
  UNIT_TAIL = 1,        // block-scaled, full tiles elsewhere: the one unit is the partial last tile
  UNIT_ROWS = 2,        // groups of 8..256 elements, no power of two >= 32: unit u is the groups u * slot .. u * slot + slot - 1
  UNIT_PLAIN_BF16 = 3,  // unquantized: unit u is tile u
  UNIT_PLAIN_FP32 = 4,
  UNIT_ROW = 6,         // groups of 264..512 elements of that kind: unit u is group u
  UNIT_WIDE = 5         // groups of 520..8192 elements: a workgroup's unit, see wide_geometry
};

// Tensor-wise scaling in one pass (eco_step_resident_kernel): slabs of one 512-element tile to each of a workgroup's 12
// waves, five of them in hand.  Three waves of 168 registers fill a SIMD's 512 (INT4, 369 M elements, us: 12 waves 940 and 16 with
// four slabs of 128 registers 957; an earlier form 1000, and 8 with eight of 256 registers 1290).
constexpr int RES_WAVES = 12, RES_DEPTH = 5;
constexpr uint64_t RES_SLAB = static_cast<uint64_t>(RES_WAVES) * TILE_ELEMS;
// Slabs a tensor may have for each workgroup: the exchange of maxima takes two of the turns in hand.
constexpr uint64_t RES_SLABS_PER_WG = RES_DEPTH - 2;
// Bytes of a tensor's arrays, each counted once: whether a step finds them in the 256 MB cache in front of HBM decides
// which form of it is the faster one.
struct StateLayout { bool adam, state_bf16, aux, master = false; };      // aux: a stored error or master weights
inline uint64_t array_bytes(uint64_t numel, int fmt, const StateLayout &l) {
  const bool quantized = fmt == FMT_FP8 || fmt == FMT_INT4;
  const uint64_t half = fmt == FMT_FP8 ? 2 : fmt == FMT_INT4 ? 1 : fmt == FMT_BF16_PLAIN ? 4 : 8;      // of the weights, in half bytes
  return numel * (2 + (l.adam ? 2 : 1) * (l.state_bf16 ? 2 : 4) + (l.aux && quantized ? 4 : 0)) + numel * half / 2;
}
// Whether the tensor-wise tensors of one format that the chip can hold are stepped in one pass.  In favour: 35 % fewer bytes (10 to 15 %
// with master weights, whose second pass reads them alone), and two launches where the two-pass form has four.  Against: turns of 4 to 5 us, so
// that lists of few turns (but more than one) are slower; a launch of 5 us more where a tensor has a tail; two launches more where longer
// tensors need the two-pass form anyway.  The lines are where the two forms met, by the bytes of the tensors that one pass would take (tensors
// of 300 000 elements; us, two passes / one) --
//   one turn: Adam, fp32 state 15.4 / 13.3 (1.2 M elements).
//   fp32 state and a stored error: Adam 30.6 / 31.6 (53 MB), 42.2 / 35.2 (79); SGDM 20.9 / 21.8 (34), 27.5 / 26.6 (50), 33.2 / 35.0 (67), 59.8 / 49.6.
//     Tails: Adam 41.7 / 41.3 (79), 52.7 / 52.3 (106), 92.5 / 76.6; SGDM 33.0 / 39.1 (67), 59.9 / 54.7 (134).  Beside a longer tensor: Adam 124.8 /
//     128.3 (211), 233.8 / 212.5 (422); SGDM 76.1 / 78.5 (134), 134.8 / 118.7 (269); stored error 111 / 113 (211), 208 / 200 (422).
//   bf16 state, Adam: INT4 35.3 / 38.6 (62), 59.1 / 57.9 (125); FP8 36.6 / 39.1 (67), 62.9 / 58.0 (134).  Tails: 59.0 / 64.2 (125), 104.2 / 101.8
//     (250); FP8 62.4 / 64.3 (134), 114.3 / 106.5 (269).  Beside a longer one: 123.5 / 133.1 (250), 249 / 224 (499); FP8 134.7 / 136.4 (269).
//   bf16 state, SGDM, the fewest bytes: 71.0 / 73.8 (173), 140.1 / 137.3 (346), with tails 139.8 / 145.0.
//   master weights, Adam, fp32 state: 32.2 / 33.6 (72), 43.3 / 38.5 (108), bf16 state 25.5 / 29.7 (50), 34.2 / 33.3 (76).  Tails 111.8 / 112.1 (288),
//     215.6 / 223.4 (576), 434 / 422 (1152).  Beside a longer one 248 / 264 (576), 466 / 462 (1152).  SGDM 24.9 / 26.6 (53), 33.9 / 30.3 (79); tails
//     42.2 / 43.4 (106), 72.8 / 66.5 (211), 146 / 158 (422), 317 / 299 (845); beside a longer one 173 / 193 (422), 332 / 330 (845).
inline bool one_pass_pays(const StateLayout &l, uint64_t bytes, uint64_t slabs, unsigned cus, bool tails, bool beside_longer) {
  if (slabs <= cus && !tails && !beside_longer) return true;
  enum { F32_ADAM, F32_SGDM, BF16_ADAM, BF16_SGDM, MASTER_ADAM, MASTER_SGDM };
  constexpr uint64_t from_mb[][4] = {{56, 96, 224, 260}, {48, 96, 200, 228}, {100, 208, 320, 416}, {384, 384, 384, 384}, {80, 800, 1100, 1100},
                                     {64, 130, 1000, 1000}};
  const int row = l.master ? (l.adam ? MASTER_ADAM : MASTER_SGDM) : !l.state_bf16 || l.aux ? (l.adam ? F32_ADAM : F32_SGDM) : l.adam ? BF16_ADAM : BF16_SGDM;
  return bytes >= 1000000 * from_mb[row][(tails ? 1 : 0) + (beside_longer ? 2 : 0)];
}
// Workgroups of the finishing kernel: a wave to each tensor, for its scale, and where waits may be given up enough for the
// slabs that are then marked, a workgroup to each up to four per compute unit (they return after one load where none is:
// 12.9 us for three tensors of 40 000 elements with one workgroup and with 21, 34 us for one of 4.7 M with 1 and with 768).
// With elementwise kernels of another stream on the chip a step of 4.7 M elements takes 0.28 ms, and took 4.0 when
// one workgroup finished them all; of 92 M 1.17 ms, and 9.2.
constexpr unsigned RES_FINISH_THREADS = 256;
inline unsigned res_finish_workgroups(uint64_t tensors, uint64_t slabs, unsigned cus) {
  constexpr uint64_t waves = RES_FINISH_THREADS / 64;
  const uint64_t most = 4ull * cus, for_tensors = (tensors + waves - 1) / waves;
  const uint64_t wgs = slabs > for_tensors ? slabs : for_tensors;
  return static_cast<unsigned>(wgs < most ? wgs : most);
}
constexpr uint32_t RES_TRIES = 64;           // reads of slab_max[] before a wait is given up, 1.5-2 us each

struct TensorDesc {          // 80 bytes, device table entry
  void *w;                   // weights / codes
  void *s;                   // scales
  const void *g;             // bf16 gradient
  void *m;
  void *v;
  void *aux;                 // fp32: stored error (exact injection) or master weights
  uint64_t numel;
  uint64_t group_size;       // elements per scale group
  uint32_t first_unit;       // index of this tensor's first unit (tile, group, bundle of groups) in its launch list
  uint32_t tensor_id;
  uint16_t bs_shift;         // log2(group_size) for power-of-two groups of 32..512 elements
  uint16_t kind;             // UNIT_*: what a unit of the list the tensor is in stands for
  uint32_t slot;             // tensor-wise scaling: index of the tensor's abs-max slot; in one pass: elements beyond numel, which
                             // is a multiple of 8 there; wide groups and UNIT_ROWS: groups per unit
};
static_assert(sizeof(TensorDesc) == 80, "TensorDesc layout");

struct StepArgs {            // by-value kernel argument: everything wave-uniform
  const TensorDesc *tensors;
  const uint32_t *extra_tensor;    // one-wave units that ride in this launch: unit -> index into tensors
  const uint32_t *tw_tile_tensor;  // tensor-wise scaling: tile (full or partial) -> index into tensors
  const uint32_t *tw_tensor;       //   ... the tensors themselves
  uint32_t *slots;                 //   ... one abs-max slot (fp32 bit pattern) per such tensor
  uint32_t *tile_max;              //   ... scratch: the abs-max of every such tile, written and consumed within a step
  const uint32_t *slab_tensor;     // tensor-wise scaling in one pass: slab -> index into tensors
  uint32_t *slab_max;              //   ... scratch: each slab's abs-max, all ones until it is known; empty again after the step
  const uint32_t *resident_tensor; //   ... the tensors themselves
  uint32_t *deferred;              //   ... scratch: which slabs are left to the finishing kernel (0 or 1 each)
  uint32_t *tail_max;              //   ... scratch: abs-max of the tensors' tails, by place in resident_tensor
  uint32_t *resident_counts;       //   ... scratch: whether there are any; workgroups through with them
  uint32_t resident_wgs;           //   ... workgroups of the launch in flight
  uint32_t num_tiles, num_extra, num_tw_tiles, num_tw_tensors, num_slabs, num_resident, resident_tails, resident_tries;
  uint32_t tw_reduce_wgs;          // tensor-wise scaling: workgroups per tensor of the reduction
  float b1, omb1, b2, omb2, rbc2, c1, eps, kappa, lr, alpha, wd, inv_lr, inv_lr_beta;
  uint32_t seed_lo, seed_hi, step_lo;
  uint32_t div_mid;                // c1 and eps allow the short division (see div_rn_midrange) after a short square root
  uint32_t unit_base;              // first work item (group, tile, tensor) of the launch in flight, see launch_in_chunks
  uint32_t num_units;              // wide-group launch: work items before the extra ones
  uint32_t wg_waves;               // waves of a workgroup of the launch in flight (a kernel that asks the runtime for its geometry is
                                   // passed 256 bytes of arguments more, 0.7 to 1 us of a call)
};

// A list of at most SMALL_TENSORS tensors, carried by value in the kernel arguments (4 KB): the allocation-free step of a short
// list needs no table in device memory and is one launch whatever classes of scale group it holds.
constexpr int SMALL_TENSORS = 44;
struct SmallArgs {
  StepArgs step;
  uint32_t num;                        // tensors
  uint32_t first_wg[SMALL_TENSORS];    // the first workgroup of each
  TensorDesc desc[SMALL_TENSORS];
};
static_assert(sizeof(SmallArgs) <= 4096, "kernel arguments are limited to 4 KB");

inline uint32_t tw_reduce_workgroups(uint64_t most_tiles) {
  const uint64_t w = (most_tiles + 16383) / 16384;
  return static_cast<uint32_t>(w < 1 ? 1 : w > 64 ? 64 : w);
}

constexpr int STREAM_TENSORWISE = MAX_WIDE_WAVES + 1;

// What one format's step launches, host side.
struct StepLaunch {
  StepArgs args;
  uint64_t max_launch_threads;     // most threads one launch may have (the runtime's limit, or a smaller one set for tests)
  uint64_t max_tile_threads;       // the same for the full-tile kernel (a tuning option may cap it further)
  uint32_t lds_bytes;              // dynamic LDS per workgroup of the full-tile kernel (occupancy cap)
  uint32_t lds_bytes_wide[MAX_WIDE_WAVES + 1];   // the same per workgroup of the wide-group kernel, by its waves
  uint32_t lds_bytes_tw;           // the same per (one-wave) workgroup of the two tensor-wise passes
  const uint32_t *tile_tensor;     // block-scaled tensors: full tile -> index into the descriptors; args.extra_tensor lies behind it
  const uint32_t *list_tensor;     // the list kernel: workgroup -> index into the descriptors
  const uint32_t *wide_base;       // group -> index into the descriptors: wide-group lists, one per workgroup size, back to back
  uint32_t wide_offset[MAX_WIDE_WAVES + 1];
  uint32_t num_wide[MAX_WIDE_WAVES + 1];
  unsigned resident_wgs;           // workgroups of the one-pass tensor-wise kernel: one per compute unit
  uint32_t stream;                 // which launches pass the caches by (see stream_launches), a bit each: 0 the full-tile one, n the wide groups of n
                                   // waves, STREAM_TENSORWISE the long tensors with one scale
  int extra_in;                    // which launch the one-wave units ride in: 0 the full-tile one, n the wide groups of n waves
  const SmallArgs *small;          // if set, one launch of eco_step_small_kernel (arguments by value),
  uint64_t list_wgs;               // or if not 0, of the list kernel,
  unsigned list_waves;             //   with workgroups of so many waves, stands for all of the above but the tensor-wise passes
};

struct KernelVariant {
  int fmt;          // FMT_*
  int state_bf16;   // m, v stored as bfloat16
  int scale_bf16;
  int algo;         // ALGO_*
  int round;        // ROUND_*
};

// Each launcher enqueues its kernels on `stream`, checks every launch, and returns the first error.
hipError_t launch_step(const KernelVariant &kv, const StepLaunch &sl, hipStream_t stream);
hipError_t launch_quantize_init(const void *src, int src_bf16, uint64_t numel, int fmt, uint64_t group_size,
                                int scale_bf16, void *weights, void *scales, hipStream_t stream);
hipError_t launch_dequantize(const void *weights, const void *scales, uint64_t numel, int fmt, uint64_t group_size,
                             int scale_bf16, const void *src, int src_kind, float *dst, hipStream_t stream);

hipError_t launch_bandwidth_probe(int kind, void *codes, void *scales, const void *grad, void *m, void *v, uint64_t numel, bool streamed,
                                  uint32_t lds_bytes, hipStream_t stream);

hipError_t launch_arith_selftest(int kind, float numerator, uint32_t bits_lo, uint32_t bits_hi, unsigned long long *mismatches,
                                 hipStream_t stream);

// Scale-group classes (how the abs-max of a group is reduced)
enum : int { GROUP_BLOCK = 0, GROUP_WIDE = 1, GROUP_TENSOR = 2, GROUP_UNSUPPORTED = -1 };
inline int classify_group(uint64_t group_size, uint64_t numel) {
  if (group_size >= 32 && group_size <= 512 && (group_size & (group_size - 1)) == 0) return GROUP_BLOCK;
  const uint64_t g = group_size < numel ? group_size : numel;       // a group never exceeds the tensor
  if (g <= MAX_WIDE_GROUP && g % 8 == 0) return GROUP_WIDE;
  if (group_size >= numel) return GROUP_TENSOR;
  return GROUP_UNSUPPORTED;
}
// The helper kernels (initial quantizer, de-quantizer, error) take one launch with one workgroup per tile or per
// wide group, and the runtime wants grid x block below 2^32: about 2^35 elements a call.
constexpr uint64_t MAX_LAUNCH_THREADS = 0xFFFFFFFFull;
inline bool flat_call_fits(uint64_t numel, uint64_t group_size) {
  if (numel > (1ull << 40)) return false;
  uint64_t threads = (numel + TILE_ELEMS - 1) / TILE_ELEMS * WG_THREADS;
  if (classify_group(group_size, numel) == GROUP_WIDE) {
    const uint64_t g = group_size < numel ? group_size : numel;
    threads = (numel + g - 1) / g * 64 * ((g + TILE_ELEMS - 1) / TILE_ELEMS);
  }
  return threads <= MAX_LAUNCH_THREADS;
}
// A flat kernel with 8 elements to a thread: its workgroups, and how many of them one launch may have.  A helper call
// of the largest size that flat_call_fits lets through is 2^32 - 64 threads; rounded up to whole workgroups of more than
// 64 threads it is 2^32, one launch too many, so those kernels are told the first workgroup of each launch.
struct FlatLaunch { uint64_t workgroups, per_launch; };
inline FlatLaunch flat_launch(uint64_t numel, unsigned threads) {
  const uint64_t share = static_cast<uint64_t>(threads) * ELEMS_PER_LANE;
  return {(numel + share - 1) / share, MAX_LAUNCH_THREADS / threads};
}
// Wide groups (a multiple of 8 up to 8192 elements, not a power of two in [32, 512]): one workgroup of `waves` waves
// takes `rows` consecutive groups.  One group a workgroup in general; groups of more than 512 elements whose length is
// not a multiple of 512 leave lanes of their last wave idle, so where 2..8 of them together fill a whole number of
// waves exactly (1408 = 2.75 waves: four rows in 11 waves; 576: eight rows in 9 waves) and the tensor is a whole number
// of such bundles, a workgroup takes the bundle.  This is the initial quantizer's grouping, that of steps of less than 96 MB of arrays (of
// less than 384 MB where the other takes more launches), of steps of Adam with master weights, and of allocation-free calls whose tables hold no
// other; for the others see step_geometry.
struct WideGeometry { uint32_t rows; uint32_t waves; uint64_t units; };
inline WideGeometry wide_geometry(uint64_t numel, uint64_t g) {          // g = min(group size, numel)
  const uint64_t ngroups = (numel + g - 1) / g;
  WideGeometry w = {1u, static_cast<uint32_t>((g + TILE_ELEMS - 1) / TILE_ELEMS), ngroups};
  if (g > TILE_ELEMS && g % TILE_ELEMS != 0 && numel % g == 0) {
    for (uint32_t k = 2; k <= 8; ++k) {
      if ((k * g) % TILE_ELEMS == 0 && k * g / TILE_ELEMS <= MAX_WIDE_WAVES && ngroups % k == 0) {
        w.rows = k;
        w.waves = static_cast<uint32_t>(k * g / TILE_ELEMS);
        w.units = ngroups / k;
        break;
      }
    }
  }
  return w;
}
// How steps of 96 MB of arrays and more group them.  A step's waves tolerate idle lanes (see WavePieces), and what a large workgroup costs
// is more: its waves wait for the slowest, and come and go together.  So few waves, most of their lanes busy: two to four rows whose
// last wave may be part idle, the last workgroup of a tensor with what rows there are.  Measured over 150 M elements, each
// with the best number of resident waves, us: one row / this / the bundle that fills its waves exactly --
//   fp32 state, Adam: 576 543 / 510 / 513 (3 rows in 4 waves), 640 561 / 510 / 515, 896 544 / 519 (4 in 7), 1152 513 / 512 / 516 (2
//   in 5), 1408 507 (one) / 548, 2304 513 (one) / 517, 2816 512 (one) / 555; SGDM: 576 327 / 305 / 308, 1152 305 / 302 / 307, 1408 303
//   (one) / 311; SGDM with master weights 1152 509 / 490 / 522.
//   bf16 state, Adam, INT4: 576 389 / 307 / 312, 640 357 / 295 / 294, 896 303 / 293.  Without a cap on resident waves, which most rows with
//   idle lanes of this kind do not have, the exact bundle otherwise: 1408 315 / 313 (FP8 344 / 322), 2304 310 / 303, 2816 315 / 307;
//   longer ones lose (1664 304 / 330 in 13 waves).
//   Adam with master weights, without such a cap: the exact bundle (576 790 / 764, 640 785 / 740, 1152 752 /
//   762, 2304 767 / 770).  (With the cap that longer steps have, see wide_workgroups_idle, other bundles may be the better ones; not measured.)
// Where it is all but as good and of up to 9 waves the exact bundle stays: row lengths that share a number of waves share a launch
// (510 M elements in rows of 576 and of 2304, all in 9 waves 1833 us, in 4 and in 5 1843).
inline WideGeometry step_geometry(uint64_t numel, uint64_t g, const StateLayout &l) {        // g = min(group size, numel)
  const uint64_t ngroups = (numel + g - 1) / g;
  const WideGeometry exact = wide_geometry(numel, g);
  const bool pair = !l.state_bf16 && g > 2 * TILE_ELEMS && 2 * g <= 5 * TILE_ELEMS;
  if ((l.aux && l.adam) || (exact.rows > 1 && !pair && exact.waves <= (l.state_bf16 ? 11 : 9))) return exact;
  uint64_t k = 1;
  if (g <= TILE_ELEMS) k = 1;
  else if (3 * g <= 4 * TILE_ELEMS) k = 3;
  else if (pair || 2 * g <= 3 * TILE_ELEMS) k = 2;
  else if (4 * g <= 7 * TILE_ELEMS) k = 4;
  if (k > ngroups) k = ngroups;
  return {static_cast<uint32_t>(k), static_cast<uint32_t>((k * g + TILE_ELEMS - 1) / TILE_ELEMS), (ngroups + k - 1) / k};
}
// Whether the initial quantizer takes the bundle too.  It moves a third of the step's bytes and is the sooner bound by the
// longer workgroup's waves coming and going together: four rows or more to a workgroup pay where a row alone leaves at least an
// eighth of its lanes idle, with INT4 codes a fifth (100 M elements, us, one row / the bundle: FP8 rows of 1152 126 / 121, 1664
// 121 / 118, 1408 117 / 123, 1920 117 / 123; INT4 from bf16 1152 103 / 98, 1664 94 / 96, 1408 87 / 96, 1920 84 / 88), two rows always
// (2816 127 / 120 and 102 / 92).
inline bool quantizer_takes_bundle(uint32_t rows, uint64_t g, int fmt) {
  const uint64_t lanes = (g + TILE_ELEMS - 1) / TILE_ELEMS * TILE_ELEMS;
  return rows == 2 || (rows > 2 && (lanes - g) * (fmt == FMT_INT4 ? 5 : 8) >= lanes);
}
// Groups of up to 512 elements that are no power of two in [32, 512] (rows of 48, 96, 384, ...): as many whole groups to
// a wave as its 512 elements hold (one from 264 on).
inline uint32_t rows_per_wave(uint64_t g) { return static_cast<uint32_t>(TILE_ELEMS / g); }

// What a step does with one tensor: the launch list it enters, the kind of its units there and how many they are.
enum : int { LIST_TILE = 0, LIST_EXTRA = 1, LIST_WIDE1 = 2, LIST_TW_TILES = LIST_WIDE1 + MAX_WIDE_WAVES, LIST_RESIDENT, LIST_COUNT };
struct Placement {
  int list;              // LIST_*; LIST_WIDE1 + n - 1: groups that take a workgroup of n waves
  int kind;              // UNIT_*
  uint64_t units;
  bool tail;             // one more unit, of kind UNIT_TAIL, in LIST_EXTRA
  uint64_t group;        // elements per scale group
  uint32_t rows;         // groups per unit (wide groups, UNIT_ROWS)
  bool idle;             // wide groups: the units leave lanes of their last wave idle
  uint64_t entries;      // what the tensor counts towards the limits on launch tables: a unit per tile or per group
};
// slab, max_slabs: the one-pass tensor-wise kernel's slab length and the most slabs of a tensor it may take (0: none).
// step: of a step (null: for the initial quantizer, which shares the grouping of rows); own_rows: with the step's own grouping.
struct StepRows { StateLayout layout; bool own_rows; };
// (inlined always: the allocation-free call places every tensor twice, and 40 of them take 0.1 us less so)
__attribute__((always_inline)) inline Placement place_tensor(uint64_t numel, uint64_t group_size, int cls, bool quantized, int fmt,
                                                             uint64_t slab = TILE_ELEMS, uint64_t max_slabs = 0, const StepRows *step = nullptr) {
  Placement p = {LIST_TILE, UNIT_TILES, 0, false, group_size, 1, false, 0};
  if (cls == GROUP_BLOCK) {
    const bool rest = numel % TILE_ELEMS != 0;
    p.entries = numel / TILE_ELEMS + (rest ? 1 : 0);
    if (!quantized) {
      p.list = LIST_EXTRA;
      p.kind = fmt == FMT_BF16_PLAIN ? UNIT_PLAIN_BF16 : UNIT_PLAIN_FP32;
      p.units = p.entries;
    } else {
      p.units = numel / TILE_ELEMS;
      p.tail = rest;
    }
  } else if (cls == GROUP_WIDE || (step && numel <= MAX_WIDE_GROUP)) {
    // (one scale for a whole tensor of up to 8192 elements is one group, of any length: its last piece of 8 elements is cut off; 282
    // tensors of 64, 318 and 2650 elements, us: those of odd length in slabs, with a launch for their tails, 17.0, so 6.2)
    p.group = group_size < numel ? group_size : numel;
    if (p.group <= static_cast<uint64_t>(TILE_ELEMS)) {
      p.list = LIST_EXTRA;
      p.rows = cls == GROUP_WIDE ? rows_per_wave(p.group) : 1;
      p.kind = p.rows > 1 ? UNIT_ROWS : UNIT_ROW;
      p.entries = (numel + p.group - 1) / p.group;
      p.units = (p.entries + p.rows - 1) / p.rows;
    } else {
      WideGeometry w = wide_geometry(numel, p.group);
      p.entries = w.units;
      if (step && step->own_rows) w = step_geometry(numel, p.group, step->layout);
      p.list = LIST_WIDE1 + static_cast<int>(w.waves) - 1;
      p.kind = UNIT_WIDE;
      p.rows = w.rows;
      p.units = w.units;
      p.idle = w.rows * p.group % TILE_ELEMS != 0;
    }
    if (cls == GROUP_TENSOR) p.entries = (numel + TILE_ELEMS - 1) / TILE_ELEMS + 1;
  } else {
    p.group = numel;
    p.list = LIST_TW_TILES;
    p.units = (numel + TILE_ELEMS - 1) / TILE_ELEMS;
    p.entries = p.units + 1;
    // one pass where the chip can hold the tensor (its lanes have 8 elements or none; up to 7 last ones are a tail)
    const uint64_t whole = numel / ELEMS_PER_LANE * ELEMS_PER_LANE, slabs = whole <= slab ? 1 : (whole + slab - 1) / slab;
    if (slabs <= max_slabs) {
      p.list = LIST_RESIDENT;
      p.units = slabs;
    }
  }
  return p;
}
// Workgroups of `nw` waves of the wide-group kernel to have resident per compute unit (0: as many as fit), for arrays that
// come from HBM (see HbmBound).  HBM delivers most with a certain amount of traffic in flight; more waves only add latency.
// So the smallest number of workgroups with at least that many waves' worth of busy lanes --
// (a) where the lanes are busy, us, 150 M elements, with / without:
//   Adam, fp32 state: 12 waves, as the full-tile kernel (fill_step_scalars).
//   Adam, bf16 state, 20: FP8 rows of 768 309 / 337, 1024 314 / 329, 2048 323 / 337, 4096 311 / 323 (INT4 286 / 309, 294 / 305, 293 /
//   304, 290 / 303).  Workgroups of 5 to 7 and of 9 to 16 waves gain nothing or lose: 640 314 / 309, 3072 316 / 314, 8192 336 / 336.
//   Master weights, fp32 state, two or up to 10 waves: 768 701 / 789, 1024 766 / 803, 2048 724 / 793, 640 724 / 780, 4096 757 / 771.
//   Master weights, bf16 state, 12: 1024 478 / 519, 2048 505 / 546, 3072 505 / 533.
//   SGDM, fp32 state, 14.5: 768 304 / 328, 1024 310 / 319, 2048 299 / 332, 3072 301 / 332, 3584 302 / 338, 4096 314 / 332 (larger
//   workgroups lose: 2304, two of 9 waves, 332 / 309); with a stored error, 11.5: 768 510 / 551, 1024 511 / 525, 2048 501 / 527, 4096 531 / 537; with master weights, 8.5: 768 489 /
//   529, 1024 507 / 521, 2048 511 / 541, 4096 515 / 532.
// streamed: where the launch passes the caches by (us, the others' / these: Adam, fp32 state, rows of 1024 180 / 174, 2048 544 / 470; with master
// weights 1024 466 / 446).
inline unsigned wide_workgroups(const KernelVariant &kv, unsigned nw, bool streamed = false) {
  const auto at_least = [nw](unsigned tenths) { const unsigned k = (tenths + 10 * nw - 1) / (10 * nw); return k < 2 ? 2 : k; };
  if (streamed && !kv.state_bf16 && algo_is_adam(kv.algo)) return at_least(kv.algo == ALGO_ADAM ? 120 : 80);
  if (kv.algo == ALGO_ADAM) return kv.state_bf16 && (nw <= 4 || nw == 8) ? at_least(200) : 0;
  if (kv.algo == ALGO_ADAM_MASTER) return kv.state_bf16 ? at_least(115) : nw <= 5 ? 10 / nw : 2;
  if (kv.state_bf16) return 0;
  if (kv.algo == ALGO_SGDM) return nw <= 8 ? at_least(145) : 0;
  return at_least(kv.algo == ALGO_SGDM_EXACT ? 115 : 85);
}
// (b) where rows leave lanes idle, `elements` in the launch's `units` workgroups of `nw` waves (150 M elements, with / without, if not said
// otherwise):
//   Adam, fp32 state, 13.6: 520 523 / 590, 640 510 / 577, 1000 522 / 629, 1152 512 / 520, 1408 510 / 575, 1800 515 / 608, 2304 513 /
//   527, 2816 512 / 545, 3000 519 / 596, 3328 521 / 557, 4000 511 / 612 (INT4 1000 510 / 586, 1800 485 / 566, 3000 490 / 567).
//   Adam, bf16 state, workgroups of up to 4 and of 8 waves of which nineteen lanes in twenty are busy, from 600 MB on, in INT4 from 1 GB, 19.5:
//   FP8 620 MB 1000 203 / 212, 1480 197 / 205, 2000 193 / 201, 2.8 GB 760 879 / 973, 1000 865 / 1012, 2000 854 / 982, 4000 850 / 905; INT4 1.4 GB 760 449 /
//   464, 1000 446 / 477, 2000 433 / 459 (620 MB 760 212 / 199, 1000 200 / 208).  Others lose: 2528 in workgroups of 5 891 / 857, rows with
//   fewer lanes busy (1344, INT4 620 MB) 197 / 188.
//   Master weights, fp32 state, from 600 MB on, 9.5: FP8 620 MB 1000 204 / 221, 1344 198 / 216, 1800 203 / 226, 3000 208 / 218, 2.8 GB 966 /
//   1179, 867 / 1056, 916 / 1131, 920 / 1107, 1152 872 / 941, 1408 876 / 960; of 4000 and longer two workgroups are more than that already.
//   Master weights, bf16 state, 11.5: 1000 529 / 641, 1408 494 / 541, 1800 531 / 600, 2816 494 / 529.
//   SGDM, fp32 state, 19.6: 640 302 / 338, 1152 302 / 305, 1408 306 / 321; FP8 1.4 GB (22 waves' worth / this) 760 441 / 426, 1000 467 / 452, 1344
//   443 / 422, 1800 458 / 413, 5000 412 / 412; with a stored error, 15.6: 640 531 / 545, 1152 529 / 547, 1408 540 / 568, 3000 546 / 571; 1.4 GB
//   (16.5 waves' worth / this) 1000 466 / 443, 1344 461 / 440, 4000 488 / 448; with master weights, 9.7: 640 486 / 538, 1000 514 / 631, 1152
//   490 / 534, 1408 496 / 525, 1800 506 / 607, 2304 494 / 538, 3000 527 / 609.
//   SGDM, bf16 state, with master weights 13.6, INT4 1.2 GB (FP8 alike): 520 355 / 385, 576 368 / 397, 640 356 / 390, 760 360 / 401, 1000 377 /
//   449, 1496 387 / 423, 1800 360 / 399, 2304 354 / 372, 3000 353 / 397, 4000 366 / 398, 6912 370 / 370 (390 MB: 520 126 / 114, 1000 113 / 115, 3000
//   113 / 118); with a stored error 20.4: 576 364 / 365, 760 359 / 380, 1000 371 / 403, 1408 368 / 377, 1496 377 / 405, 1800 362 / 373, 2304 371 / 371.
// Adam with fp32 state and SGDM with a stored error, where rows start off the lines of memory and are not streamed (1.6 GB of arrays, 13.6 and
// 15.6 / this): 11.5 544 532 / 498, 560 556 / 512, 1000 524 / 501, 2016 517 / 490, in the cache 1152 66.4 / 64.8; 11.8 1000 552 / 500, 2016 514 / 505.
// The other figures are from before waves took whole lines at a time (see exchange_chunks).  Since then, rows that start off the lines of memory,
// 460 MB and 1.4 GB of arrays, us, as above / as now: SGDM, bf16 state, with a stored error (20.4 / 15) FP8 1000 153 / 138, 497 / 417, 3000 149 / 139,
// 475 / 419, INT4 2024 154 / 138, 490 / 409; fp32 state, FP8, where fewer than nine lanes in ten are busy (19.6 / 17) 544 143 / 138, 445 / 409; INT4 with
// a stored error from 1 GB (11.8 / 11.2) 1480 467 / 435, 3000 491 / 443 (1000 424 / 431); with master weights (9.7 / 10.6) 1000 150 / 143, 448 / 429;
// Adam, master weights (9.5 / 8.5) 1.4 GB 760 516 / 462, 1480 485 / 450; Adam, in part in the cache (11.5 / 13) 1480 330 MB 103.1 / 98.2.
inline unsigned wide_workgroups_idle(const KernelVariant &kv, uint64_t bytes, unsigned nw, uint64_t units, uint64_t elements,
                                     bool streamed = false) {
  const auto at_least = [=](uint64_t tenths) {
    const uint64_t k = (tenths * units * TILE_ELEMS + 10 * elements - 1) / (10 * elements);
    return static_cast<unsigned>(k < 2 ? 2 : k);
  };
  const uint64_t MB = 1000000;
  const bool fp8 = kv.fmt == FMT_FP8, long_step = bytes >= 600 * MB, nearly_all = (nw <= 4 || nw == 8) && elements * 20 >= units * nw * TILE_ELEMS * 19;
  switch (kv.algo) {
    case ALGO_ADAM:
      if (!kv.state_bf16) return at_least(streamed ? 136 : bytes >= 384 * MB ? 115 : 130);
      return nearly_all && bytes >= (fp8 ? 600 : 1000) * MB ? at_least(195) : 0;
    case ALGO_ADAM_MASTER: return kv.state_bf16 ? at_least(115) : long_step ? at_least(streamed ? 95 : 85) : 0;
    case ALGO_SGDM: return kv.state_bf16 ? 0 : at_least(fp8 && !streamed && elements * 10 < units * nw * TILE_ELEMS * 9 ? 170 : 196);
    case ALGO_SGDM_EXACT: return at_least(kv.state_bf16 ? 150 : streamed ? 156 : fp8 || bytes < 1000 * MB ? 118 : 112);
    default: return at_least(kv.state_bf16 ? 136 : 106);
  }
}
// Waves per compute unit of a launch of one-wave units alone (short rows), `elements` in `units` of them; 0: as many as fit.
// Again the smallest number with a certain number of waves' worth of busy lanes.  For arrays that come from HBM, 100 M elements,
// us, with / without --
//   (Before waves took whole lines at a time, see exchange_chunks.  Since then those that pass the caches by, fp32 state, Adam 13.4 instead of 10.3,
//   1.6 GB 192 510 / 471, 384 500 / 476; master weights 9 instead of 7, 192 508 / 479, 384 498 / 481; a stored error 12 instead of 13.4, 384 485 / 462;
//   SGDM with master weights 10.5 instead of 8.2, 460 MB 192 157 / 136.  And those off the lines, 460 MB and 1.4 GB, the caps of the former / as now:
//   fp32 state, Adam FP8 12 264 165 / 154, 511 / 462, INT4 11 40 163 / 149, 501 / 438; master weights, where fewer than three lanes in four are busy, 8.5
//   328 1.4 GB 536 / 481; a stored error 11 504 FP8 155 / 146, 495 / 435; SGDM FP8 17.5 200 147 / 140, 435 / 414, where fewer are busy 15 from 768 MB, 328
//   458 / 432; with master weights 10.5 48 167 / 148, 496 / 447.  bf16 state, Adam 19, in FP8 from 600 MB, 40 to 504 at 450 MB and 1.6 GB 3.5 % less time
//   on average; with master weights where fewer than three in four are busy 10.5 328 169 / 154, 550 / 462, in FP8 from 600 MB for all, 48 495 / 450 (INT4
//   136 490 / 509); SGDM with master weights 12 for all, 328 166 / 149, 536 / 446; with a stored error 16, INT4 14 40 157 / 145, 502 / 431.)
//   Adam, fp32 state, 10.3: rows of 48 369 / 389, 160 368 / 393, 200 365 / 391, 328 378 / 395, 400 362 / 406, 504 393 / 415 (INT4 354 / 368,
//   353 / 372, 359 / 370, 361 / 373, 355 / 383, 366 / 395); bf16 state, 20.5, where nine lanes in ten are busy: INT4 48 214 / 219, 160
//   217 / 225, 504 211 / 229 (FP8 227 / 238, 234 / 245, 223 / 252), others none (400 243 / 222).
//   Master weights, fp32 state, 7: 96 506 / 559, 160 517 / 551, 200 544 / 590, 264 583 / 612, 328 532 / 589, 400 533 / 586, 504 535 / 599.
//   SGDM, fp32 state, 15.5, where three in four are: 48 215 / 234, 400 217 / 232, 504 214 / 247, others none (328 241 / 226); with a stored
//   error, 13.4: 48 352 / 394, 200 364 / 399, 328 369 / 405, 400 366 / 404, 504 362 / 417; with master weights, 8.2: 48 376 / 394, 160 380 / 389,
//   200 381 / 404, 264 386 / 416, 328 372 / 399, 400 369 / 408, 504 361 / 408.
//   bf16 state beside an fp32 array, where three in four are: with master weights 12.4 (1.5 GB of arrays, Adam, FP8 / INT4: 48 518 / 557 and 556 /
//   585, 96 508 / 555 and 549 / 582, 200 502 / 550 and 538 / 552, 504 531 / 559 and 556 / 583; SGDM 96 464 / 526 and 485 / 560, 400 477 / 516 and 499 / 530,
//   504 503 / 532 and 519 / 563; 328 gains nothing), with a stored error 17.2 (96 472 / 524 and 476 / 514, 200 481 / 519 and 488 / 506, 504 490 / 547 and
//   488 / 549).  SGDM, bf16 state, from 768 MB on and where nineteen lanes in twenty are busy 21.5 (504: 437 / 488, 2.6 GB 755 / 879; 390 MB 116 / 114).
// For arrays in the cache before it only Adam with fp32 state: from 96 MB on 16 where three lanes in four are busy (8 M elements: 96 28.9 / 30.0, 400
// 29.8 / 30.6; 25 M 87.8 / 90.3, 91.5 / 93.1), with master weights 14 from 192 MB on (16 M: 48 68.4 / 71.4, 96 66.9 / 68.6, 200 69.8 / 71.5, 264
// 73.1 / 72.9, 400 68.9 / 70.2, 504 68.7 / 70.7; 23 M: 96 111.3 / 114.0, 400 115.0 / 116.3, 504 113.6 / 117.9; below no difference, 9.6 M: 96
// 42.3 / 42.6, 200 43.9 / 43.9, 400 44.2 / 44.1; Adam below 96 MB lost by it, 200 2.7 M elements 11.6 / 11.2).
inline unsigned unit_workgroups(const KernelVariant &kv, uint64_t bytes, uint64_t units, uint64_t elements, bool streamed = false) {
  const uint64_t lanes = units * TILE_ELEMS, MB = 1000000;
  const auto at_least = [=](uint64_t tenths) { return static_cast<unsigned>((tenths * lanes + 10 * elements - 1) / (10 * elements)); };
  const bool fp8 = kv.fmt == FMT_FP8, long_step = bytes >= 600 * MB, most = elements * 4 >= lanes * 3, nearly_all = elements * 20 >= lanes * 19;
  if (bytes < 384 * MB) {
    if (kv.state_bf16) return 0;
    return kv.algo == ALGO_ADAM ? (most && bytes >= 96 * MB ? at_least(160) : 0)
                                : kv.algo == ALGO_ADAM_MASTER && bytes >= 192 * MB ? at_least(140) : 0;
  }
  if (kv.state_bf16) {
    switch (kv.algo) {
      case ALGO_ADAM: return elements * 10 >= lanes * 9 ? at_least(streamed || (fp8 && !long_step) ? 205 : 190) : 0;
      case ALGO_ADAM_MASTER: return !streamed && (!most || (fp8 && long_step)) ? at_least(105) : most ? at_least(124) : 0;
      case ALGO_SGDM: return nearly_all && bytes >= 768 * MB ? at_least(215) : 0;
      case ALGO_SGDM_EXACT: return !streamed ? at_least(fp8 ? 160 : 140) : most ? at_least(172) : 0;
      default: return !streamed ? at_least(120) : most ? at_least(124) : 0;
    }
  }
  switch (kv.algo) {
    case ALGO_ADAM: return at_least(streamed ? 134 : fp8 ? 120 : 110);
    case ALGO_ADAM_MASTER: return at_least(streamed || most ? 90 : 85);
    case ALGO_SGDM:
      if (!streamed && fp8 && !nearly_all) return most ? at_least(175) : bytes >= 768 * MB ? at_least(150) : 0;
      return most ? at_least(155) : 0;
    case ALGO_SGDM_EXACT: return at_least(!streamed && (fp8 || nearly_all) ? 110 : 120);
    default: return at_least(105);
  }
}
// The dynamic LDS that keeps k workgroups resident per compute unit (0: no request); LDS is handed out in pieces of 1280
// bytes, and a workgroup has up to 128 of its own beside it.  A compute unit holds 32 waves, so 32 workgroups and more are no cap.
inline uint32_t lds_for_workgroups(unsigned k) {
  if (k == 0 || k >= 32) return 0;
  const uint32_t bytes = 163840u / k / 1280u * 1280u - 256u;
  return bytes < 65536u ? bytes : 65536u;
}
// The nth piece of `pieces` where a second pass takes what a first pass left in the caches, the last pieces first.  The hardware
// hands workgroups to the eight XCDs in turn and each XCD has an L2 of its own, so a piece keeps its place among eight: the XCD that read
// it in the first pass reads it in the second.
constexpr uint32_t backwards_on_the_same_xcd(uint32_t nth, uint32_t pieces) {
  constexpr uint32_t XCDS = 8;
  const uint32_t whole = pieces / XCDS * XCDS;
  return nth < whole ? whole - XCDS - nth / XCDS * XCDS + nth % XCDS : nth;
}
inline int log2_exact(uint64_t x) { return x && !(x & (x - 1)) ? __builtin_ctzll(x) : -1; }
hipError_t launch_philox_fill(uint64_t seed, uint64_t step, uint32_t tensor_id, uint64_t first_word, uint64_t n_words,
                              uint32_t *dst, hipStream_t stream);

// per-(fmt, state) translation units of the quantized step kernel
hipError_t launch_step_fp8_f32(const KernelVariant &, const StepLaunch &, hipStream_t);
hipError_t launch_step_fp8_bf16(const KernelVariant &, const StepLaunch &, hipStream_t);
hipError_t launch_step_int4_f32(const KernelVariant &, const StepLaunch &, hipStream_t);
hipError_t launch_step_int4_bf16(const KernelVariant &, const StepLaunch &, hipStream_t);
hipError_t launch_step_plain(const KernelVariant &, const StepLaunch &, hipStream_t);

}  // namespace eco
