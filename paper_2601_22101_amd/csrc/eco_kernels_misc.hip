// Kernels beside the fused quantized step: the unquantized ("plain") optimizer step for bf16 /
// fp32 weights, the round-to-nearest initial quantizer, the dequantizer, and the raw Philox
// stream.  They share the tile geometry and the 8-element access helpers of the step kernel.
#include <mutex>

#include "eco_step_kernel.hpp"

namespace eco {

// ------------------------------------------------------------------------ plain optimizer step
// Launches of their own for unquantized tensors: a plan without quantized ones, or one whose unquantized tensors are
// too many to ride along as one-wave units (an embedding, attention matrices).  A wave per 512-element tile.
template <int FMT, bool STATE_BF16, bool ADAM, int CP>
__global__ __launch_bounds__(WG_THREADS) void eco_plain_kernel(const StepArgs a) {
  const uint32_t tile = blockIdx.x + a.unit_base;
  const TensorDesc td = load_tensor_desc(a, load_table(a.extra_tensor, tile));
  const uint64_t tile_off = (uint64_t)(tile - td.first_unit) * TILE_ELEMS, e0 = tile_off + (uint64_t)threadIdx.x * ELEMS_PER_LANE;
  if (tile_off + TILE_ELEMS <= td.numel) plain_lane<FMT == FMT_BF16_PLAIN, STATE_BF16, ADAM, ACC_FULL, CP>(a, td, e0, 8);
  else plain_lane<FMT == FMT_BF16_PLAIN, STATE_BF16, ADAM, ACC_LANE, CP>(a, td, e0, valid_from(e0, td.numel));
}

hipError_t launch_step_plain(const KernelVariant &kv, const StepLaunch &sl, hipStream_t stream) {
#define ECO_LAUNCH(F, ST, AD)                                                                                                               \
  do {                                                                                                                                      \
    if (sl.stream & 1u)                                                                                                                          \
      ECO_CHUNKS_CHECKED((eco_plain_kernel<F, ST, AD, STREAM_WAVE>), sl.args.num_extra, WG_THREADS, sl.lds_bytes, stream, sl.args, sl.max_tile_threads); \
    else                                                                                                                                    \
      ECO_CHUNKS_CHECKED((eco_plain_kernel<F, ST, AD, CACHED>), sl.args.num_extra, WG_THREADS, sl.lds_bytes, stream, sl.args, sl.max_tile_threads); \
  } while (0)
  const int key = (kv.fmt == FMT_FP32_ID ? 4 : 0) | (kv.state_bf16 ? 2 : 0) | (algo_is_adam(kv.algo) ? 0 : 1);
  switch (key) {
    case 0: ECO_LAUNCH(FMT_BF16_PLAIN, false, true); break;
    case 1: ECO_LAUNCH(FMT_BF16_PLAIN, false, false); break;
    case 2: ECO_LAUNCH(FMT_BF16_PLAIN, true, true); break;
    case 3: ECO_LAUNCH(FMT_BF16_PLAIN, true, false); break;
    case 4: ECO_LAUNCH(FMT_FP32_ID, false, true); break;
    case 5: ECO_LAUNCH(FMT_FP32_ID, false, false); break;
    case 6: ECO_LAUNCH(FMT_FP32_ID, true, true); break;
    default: ECO_LAUNCH(FMT_FP32_ID, true, false); break;
  }
#undef ECO_LAUNCH
  return hipSuccess;
}

hipError_t launch_step(const KernelVariant &kv, const StepLaunch &sl, hipStream_t stream) {
  if (kv.fmt == FMT_FP8) return kv.state_bf16 ? launch_step_fp8_bf16(kv, sl, stream) : launch_step_fp8_f32(kv, sl, stream);
  if (kv.fmt == FMT_INT4) return kv.state_bf16 ? launch_step_int4_bf16(kv, sl, stream) : launch_step_int4_f32(kv, sl, stream);
  return launch_step_plain(kv, sl, stream);
}

// ------------------------------------------------------------------------ initial quantizer
// q(x) of Sec. 3.1 with nearest-even rounding over one flat tensor, for the three classes of scale
// groups (in-wave groups, wide groups, one scale for the whole tensor in two passes).
// The two-pass form keeps its partial maxima, between its kernels, in one of QUANT_SLOTS file-scope slots; the host
// hands the slots out in turn and makes a call wait (on its own stream) for the previous user of its slot, so
// calls on different streams never share a slot that is in use.
constexpr uint64_t STREAM_BYTES = 280000000;       // from here on arrays come from HBM and go past the caches
constexpr int QUANT_SLOTS = 64, QUANT_PARTS = 256;
__device__ uint32_t g_quantize_parts[QUANT_SLOTS][QUANT_PARTS];

// Eight elements of each lane of a wave, with the cut piece if there is one: ACC_FULL or ACC_LANE (see WavePieces).  The lanes behind a
// cut piece get zeros: it may be the first of its group, and the last whole piece then one of another group's.
template <bool BF16, int ACC, int CP>
__device__ __forceinline__ void load_wave(const void *base, uint64_t e0, int nvalid, const WavePieces &wp, float (&x)[8]) {
  eco_u32x4_t q[2] = {};
  if (wp.any_whole) load_wave8<BF16, ACC == ACC_FULL, CP>(base, wp, q);
  if (wp.any_cut) {
    if (nvalid & 7) load_ragged8<BF16>(base, e0, nvalid, q);
    else if (nvalid == 0) q[0] = q[1] = eco_u32x4_t{};
  }
  unpack8<BF16>(q, x);
}

// How the quantizer's kernels load and store beside CACHED and STREAM_GROUP: a lane by itself, 32 bytes of fp32 to each.
constexpr int PER_LANE = -1;

template <int FMT, bool SCALE_BF16, bool SRC_BF16, int ACC, int RED, int CP>
__device__ __forceinline__ void quantize_lane(const void *src, void *weights, void *scales, uint64_t e0, int nvalid,
                                              uint64_t sg, int arg, bool scale_writer, int lanes = 0, uint32_t *slot = nullptr) {
  [[maybe_unused]] const WavePieces wp = ACC == ACC_FULL ? full_wave(e0) : wave_pieces(e0, nvalid);
  float x[8];
  if constexpr (CP == PER_LANE) load_state8<SRC_BF16, ACC>(src, e0, nvalid, x);
  else load_wave<SRC_BF16, ACC, CP>(src, e0, nvalid, wp, x);
  const float amax = group_absmax<RED>(absmax8(x), arg, slot, lanes);        // lanes: see there
  float s_new, inv;
  block_scale<FMT, SCALE_BF16>(amax, s_new, inv);
  uint32_t c[2];
  const Philox4 none = {0, 0, 0, 0};
  float q[8];
  encode8<FMT, ROUND_RTN, false>(x, inv, none, c, q);
  if constexpr (CP == PER_LANE) store_codes8<FMT, ACC>(weights, e0, nvalid, c);
  else store_wave_codes8<FMT, ACC, CP>(weights, e0, nvalid, wp, c);
  if (scale_writer && (ACC == ACC_FULL || nvalid > 0)) {
    if (SCALE_BF16) static_cast<uint16_t *>(scales)[sg] = (uint16_t)(f2u(s_new) >> 16);
    else static_cast<float *>(scales)[sg] = s_new;
  }
}

template <int FMT, bool SCALE_BF16, bool SRC_BF16, int CP>
__global__ __launch_bounds__(WG_THREADS) void eco_quantize_kernel(const void *src, uint64_t numel, uint32_t bs_shift,
                                                                  void *weights, void *scales) {
  const uint64_t e0 = (uint64_t)blockIdx.x * TILE_ELEMS + (uint64_t)threadIdx.x * ELEMS_PER_LANE;
  const bool writer = (threadIdx.x & ((1u << (bs_shift - 3)) - 1u)) == 0;
  if ((uint64_t)(blockIdx.x + 1) * TILE_ELEMS <= numel)
    quantize_lane<FMT, SCALE_BF16, SRC_BF16, ACC_FULL, RED_BLOCK, CP>(src, weights, scales, e0, 8, e0 >> bs_shift, (int)bs_shift, writer);
  else
    quantize_lane<FMT, SCALE_BF16, SRC_BF16, ACC_LANE, RED_BLOCK, CP>(src, weights, scales, e0, valid_from(e0, numel),
                                                                      e0 >> bs_shift, (int)bs_shift, writer);
}

// Groups of up to 512 elements that are no power of two: `rows` whole groups to a wave; ONE: one of more than 256 elements,
// reduced over the whole wave (13 M bf16 elements in rows of 264: 17.1 us with the segmented reduction).
template <int FMT, bool SCALE_BF16, bool SRC_BF16, bool ONE, int CP>
__global__ __launch_bounds__(WG_THREADS) void eco_quantize_rows_kernel(const void *src, uint64_t numel, uint32_t group_size, uint32_t rows,
                                                                       void *weights, void *scales) {
  if (ONE) {
    const uint64_t e0 = (uint64_t)blockIdx.x * group_size + (uint64_t)threadIdx.x * ELEMS_PER_LANE, end = (uint64_t)(blockIdx.x + 1) * group_size;
    quantize_lane<FMT, SCALE_BF16, SRC_BF16, ACC_LANE, RED_BLOCK, CP>(src, weights, scales, e0, valid_from(e0, end < numel ? end : numel), blockIdx.x, 9,
                                                                  threadIdx.x == 0);
    return;
  }
  const uint32_t gl = group_size >> 3, row = (threadIdx.x * (65536u / gl + 1u)) >> 16;    // lane / lanes of a group, exact below 64
  const uint64_t grp = (uint64_t)blockIdx.x * rows, e0 = grp * group_size + (uint64_t)threadIdx.x * ELEMS_PER_LANE;
  const uint64_t end = (grp + rows) * group_size;
  quantize_lane<FMT, SCALE_BF16, SRC_BF16, ACC_LANE, RED_ROWS, CP>(src, weights, scales, e0, valid_from(e0, end < numel ? end : numel),
                                                               grp + row, (int)(row * gl), threadIdx.x == row * gl, (int)gl);
}

// Wide groups: one to a workgroup, or (BUNDLE) as many as fill a whole number of waves (see quantizer_takes_bundle; two
// kernels, because the other form's code alone cost rows of 6912 up to 4 %).
template <int FMT, bool SCALE_BF16, bool SRC_BF16, bool BUNDLE, int CP>
__global__ __launch_bounds__(1024) void eco_quantize_wide_kernel(const void *src, uint64_t numel, uint32_t group_size, uint32_t rows,
                                                                 void *weights, void *scales) {
  const uint64_t grp = (uint64_t)blockIdx.x * (BUNDLE ? rows : 1), start = grp * group_size;
  const uint32_t lane_elem = threadIdx.x * ELEMS_PER_LANE;
  const uint64_t e0 = start + lane_elem;
  if (BUNDLE) {
    uint32_t row = 0;
    for (uint32_t k = 1; k < rows; ++k) row += lane_elem >= k * group_size ? 1u : 0u;
    quantize_lane<FMT, SCALE_BF16, SRC_BF16, ACC_FULL, RED_WG_ROWS, CP>(src, weights, scales, e0, 8, grp + row, (int)row,
                                                                    lane_elem == row * group_size);
    return;
  }
  const uint64_t end = start + group_size < numel ? start + group_size : numel;
  quantize_lane<FMT, SCALE_BF16, SRC_BF16, ACC_LANE, RED_WG, CP>(src, weights, scales, e0, valid_from(e0, end), grp, 0, threadIdx.x == 0,
                                                             (int)((group_size + TILE_ELEMS - 1) / TILE_ELEMS));
}

// Tensor-wise, first pass: the maximum over each workgroup's share.  One workgroup per partial maximum, which is stored, not
// merged: an atomic maximum per wave on one address took 220 us over 210 M bf16 elements.  What bounds it is the reads under way: a workgroup of
// 16 waves to a compute unit, two tiles of each wave under way, a tile's loads out again as soon as it is taken (waiting for four together, then
// loading again: 103 us; both passes of the quantizer over 250 M elements 210 -> 188, with four tiles 192, with eight more).
constexpr int QUANT_MAX_THREADS = 1024;
constexpr uint32_t QUANT_MAX_TILES = 2;
template <bool SRC_BF16, int CP>
__global__ __launch_bounds__(QUANT_MAX_THREADS) void eco_quantize_max_kernel(const void *src, uint64_t numel, uint32_t slot, uint32_t parts) {
  constexpr uint32_t WAVES = QUANT_MAX_THREADS / 64, UNDER_WAY = QUANT_MAX_TILES, CHUNKS = SRC_BF16 ? 1 : 2;
  const uint32_t stride = parts * WAVES;
  const uint64_t whole = numel / TILE_ELEMS, tiles = (numel + TILE_ELEMS - 1) / TILE_ELEMS;
  uint64_t tile = blockIdx.x * WAVES + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // Chunk k of a lane's share of a tile; fp32 needs exchange_chunks once it has arrived.
  const auto load = [&](uint64_t t, uint32_t k) {
    const eco_u32x4_t *p = static_cast<const eco_u32x4_t *>(src) + t * (64 * CHUNKS);
    return load_vec<CP>(p + (SRC_BF16 ? threadIdx.x & 63 : lane_chunk() + 64 * k));
  };
  // The maximum is one of bit patterns, as in every other reduction of the library: the float maximum would drop the NaN
  // of a lane all of whose elements are NaN.
  uint32_t amax = 0;
  const auto take = [&amax](const float (&y)[8]) { const uint32_t a = f2u(absmax8(y)); amax = amax > a ? amax : a; };
  const auto take_raw = [&take](eco_u32x4_t (&q)[2]) {
    float x[8];
    if (!SRC_BF16) exchange_chunks(q);
    unpack8<SRC_BF16>(q, x);
    take(x);
  };
  eco_u32x4_t q[UNDER_WAY][2] = {};
  const uint64_t ahead = (uint64_t)(UNDER_WAY - 1) * stride;
  if (tile + ahead < whole) {
#pragma unroll
    for (uint32_t u = 0; u < UNDER_WAY; ++u)
#pragma unroll
      for (uint32_t k = 0; k < CHUNKS; ++k) q[u][k] = load(tile + (uint64_t)u * stride, k);
    for (tile += ahead + stride; tile + ahead < whole; tile += ahead + stride) {
#pragma unroll
      for (uint32_t u = 0; u < UNDER_WAY; ++u) {           // a tile's loads go out as soon as the one before it in its registers is taken
        take_raw(q[u]);
#pragma unroll
        for (uint32_t k = 0; k < CHUNKS; ++k) q[u][k] = load(tile + (uint64_t)u * stride, k);
      }
    }
#pragma unroll
    for (uint32_t u = 0; u < UNDER_WAY; ++u) take_raw(q[u]);
  }
  for (; tile < tiles; tile += stride) {
    const uint64_t e0 = tile * TILE_ELEMS + (threadIdx.x & 63) * ELEMS_PER_LANE;
    const int nvalid = valid_from(e0, numel);
    float x[8];
    load_wave<SRC_BF16, ACC_LANE, CP>(src, e0, nvalid, wave_pieces(e0, nvalid), x);
    take(x);
  }
  __shared__ uint32_t wave_max[QUANT_MAX_THREADS / 64];
  const uint32_t w = wave_umax(amax);
  if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = w;
  __syncthreads();
  if (threadIdx.x < 64) {
    const uint32_t r = wave_umax(threadIdx.x < QUANT_MAX_THREADS / 64 ? wave_max[threadIdx.x] : 0u);
    if (threadIdx.x == 0) g_quantize_parts[slot][blockIdx.x] = r;
  }
}

// Second pass: every workgroup folds the partial maxima (its loads of them and of its elements are under way together);
// the one with the first element writes the scale.  fp32 sources backwards: the cache before HBM still holds the end of the first pass's
// reads (INT4, 80 M elements 113 us forwards, 106 backwards, 100 M 146 / 138, and with the quantization error behind it 235 / 231; up
// to 240 MB no difference).  bf16 sources forwards: 200 M elements 189 / 178, but with the error behind it 210 M 417 / 421.
template <int FMT, bool SCALE_BF16, bool SRC_BF16, int CP>
__global__ __launch_bounds__(QUANT_PARTS) void eco_quantize_tensorwise_kernel(const void *src, uint64_t numel, uint32_t parts,
                                                                              void *weights, void *scales, uint32_t slot,
                                                                              uint32_t first_wg) {
  constexpr uint64_t SHARE = (uint64_t)QUANT_PARTS * ELEMS_PER_LANE;
  const uint64_t nth = (uint64_t)first_wg + blockIdx.x, wg = SRC_BF16 ? nth : (numel + SHARE - 1) / SHARE - 1 - nth;
  const uint64_t e0 = wg * SHARE + (uint64_t)threadIdx.x * ELEMS_PER_LANE;
  const int nvalid = valid_from(e0, numel);
  const uint32_t part = threadIdx.x < parts ? g_quantize_parts[slot][threadIdx.x] : 0u;
  [[maybe_unused]] const WavePieces wp = wave_pieces(e0, nvalid);
  float x[8];
  if constexpr (CP == PER_LANE) load_state8<SRC_BF16, ACC_LANE>(src, e0, nvalid, x);
  else load_wave<SRC_BF16, ACC_LANE, CP>(src, e0, nvalid, wp, x);
  __shared__ uint32_t wave_max[QUANT_PARTS / 64];
  const uint32_t w = wave_umax(part);
  if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = w;
  __syncthreads();
  uint32_t r = wave_max[0];
#pragma unroll
  for (int k = 1; k < QUANT_PARTS / 64; ++k) r = r > wave_max[k] ? r : wave_max[k];
  float s_new, inv;
  block_scale<FMT, SCALE_BF16>(u2f(r), s_new, inv);
  uint32_t c[2];
  const Philox4 none = {0, 0, 0, 0};
  float q[8];
  encode8<FMT, ROUND_RTN, false>(x, inv, none, c, q);
  if constexpr (CP == PER_LANE) store_codes8<FMT, ACC_LANE>(weights, e0, nvalid, c);
  else store_wave_codes8<FMT, ACC_LANE, CP>(weights, e0, nvalid, wp, c);
  if (e0 == 0) {
    if (SCALE_BF16) static_cast<uint16_t *>(scales)[0] = (uint16_t)(f2u(s_new) >> 16);
    else static_cast<float *>(scales)[0] = s_new;
  }
}

// Hands out the slots of the two-pass quantizer.  A slot is free again once the second pass of its last user has run; the
// event recorded behind that kernel is what the next user of the slot waits for.
struct QuantSlotRing {
  static constexpr int MAX_DEVICES = 32;
  std::mutex mu;
  unsigned next[MAX_DEVICES] = {0};
  hipEvent_t done[MAX_DEVICES][QUANT_SLOTS] = {{nullptr}};
};
static QuantSlotRing g_quant_ring;

// Launches a kernel of `threads` threads a workgroup, whose last argument is the first workgroup of the launch.
#define ECO_FLAT_CHECKED(flat, threads, stream, kernel, ...)                                                               \
  do {                                                                                                                     \
    const FlatLaunch f_ = flat;                                                                                            \
    for (uint64_t wg_ = 0; wg_ < f_.workgroups; wg_ += f_.per_launch) {                                                    \
      const uint64_t n_ = f_.workgroups - wg_ < f_.per_launch ? f_.workgroups - wg_ : f_.per_launch;                       \
      ECO_LAUNCH_CHECKED(kernel, dim3((unsigned)n_), dim3(threads), 0, stream, __VA_ARGS__, (uint32_t)wg_);                \
    }                                                                                                                      \
  } while (0)

// Which form the quantizer's kernels take (CP).  From 280 MB of source and codes on (from fp32 320), in one pass, or from 280 MB of source on, in two
// (the second finds less in the cache before HBM), they go past the caches; not in groups of more than 4096 elements, nor from bf16 where groups fill
// their waves or share them, nor from fp32 to INT4 in rows that leave nearly half of their lanes idle.
// us, per lane / past the caches: FP8 from fp32, groups of 128, 225 MB 32.0 / 34.3, 290 42.6 / 43.0, 350 59.4 / 51.7, 600 102 / 86; rows of 1000 290 MB
// 42.9 / 44.2, 350 58.4 / 52.6, 1 GB 180 / 147, 4096 350 57.6 / 54.1, 2304 59.7 / 58.6, 170 / 164, 6912 61.1 / 62.9, 169 / 175; INT4 from fp32 760 290 MB
// 49.3 / 51.8, 350 61.8 / 61.8, 1000 43.6 / 45.3, 58.9 / 54.8, 520 77.8 / 80.9, 420 94.5 / 96.4; from bf16 2304 300 MB 75.4 / 74.0, 1000 64.8 / 59.9, 4096
// 61.9 / 63.1, 576 91.0 / 95.3.  One scale, from fp32 240 MB 76.2 / 79.7, 320 106.7 / 103.4, 520 184 / 163, from bf16 200 MB 71.7 / 79.5, 280 111.6 /
// 108.3, 500 210 / 188; with the error behind it 210 M elements from bf16 415 / 361.  What is left goes by whole pieces of a wave in rows with idle
// lanes (CACHED; from bf16, rows of 192 70 M elements 61.7 / 55.7, 1000 41.7 / 38.5), per lane elsewhere (4 M elements 4.1 / 4.2, 1152 26.5 / 27.4).
// From fp32 to INT4 also per lane in rows with a wave or up to three to themselves, and in longer ones below 40 MB (us, per lane / whole pieces: 264
// 140 MB 27.9 / 28.7, 504 22.2 / 22.7, 520 27.8 / 29.1, 576 25.4 / 26.3, 760 21.6 / 22.1, 1480 20.9 / 20.9, 6912 20 MB 4.90 / 5.14, but 60 MB 11.9 / 11.5,
// 2304 11.6 / 11.3, 4008 240 MB 36.0 / 33.6).
template <int FMT, bool SC, bool SR>
static hipError_t launch_quantize_t(const void *src, uint64_t numel, uint64_t group_size, void *weights, void *scales,
                                    hipStream_t stream) {
  const uint64_t src_bytes = numel * (SR ? 2 : 4), bytes = src_bytes + (FMT == FMT_INT4 ? numel / 2 : numel);
  const bool streamed = bytes >= (SR ? STREAM_BYTES : 320000000);
  constexpr bool INT4_F32 = FMT == FMT_INT4 && !SR;
  const uint64_t tiles = (numel + TILE_ELEMS - 1) / TILE_ELEMS;
  const int cls = classify_group(group_size, numel);
  const auto row = streamed ? eco_quantize_rows_kernel<FMT, SC, SR, true, STREAM_GROUP>
                            : eco_quantize_rows_kernel<FMT, SC, SR, true, INT4_F32 ? PER_LANE : CACHED>;
  if (cls == GROUP_BLOCK) {
    const auto kernel = streamed ? eco_quantize_kernel<FMT, SC, SR, STREAM_GROUP> : eco_quantize_kernel<FMT, SC, SR, PER_LANE>;
    ECO_LAUNCH_CHECKED(kernel, dim3((unsigned)tiles), dim3(WG_THREADS), 0, stream, src, numel, (uint32_t)log2_exact(group_size), weights, scales);
  } else if (cls == GROUP_WIDE) {
    const Placement p = place_tensor(numel, group_size, cls, true, FMT);
    if (p.kind == UNIT_ROW) {
      ECO_LAUNCH_CHECKED(row, dim3((unsigned)p.units), dim3(WG_THREADS), 0, stream, src, numel, (uint32_t)p.group, p.rows, weights, scales);
    } else if (p.kind == UNIT_ROWS) {
      const auto rows = streamed ? eco_quantize_rows_kernel<FMT, SC, SR, false, STREAM_GROUP> : eco_quantize_rows_kernel<FMT, SC, SR, false, CACHED>;
      ECO_LAUNCH_CHECKED(rows, dim3((unsigned)p.units), dim3(WG_THREADS), 0, stream, src, numel, (uint32_t)p.group, p.rows, weights, scales);
    } else if (quantizer_takes_bundle(p.rows, p.group, FMT)) {
      const auto bundle = streamed && !SR ? eco_quantize_wide_kernel<FMT, SC, SR, true, STREAM_GROUP> : eco_quantize_wide_kernel<FMT, SC, SR, true, PER_LANE>;
      ECO_LAUNCH_CHECKED(bundle, dim3((unsigned)p.units), dim3(64 * (p.list - LIST_WIDE1 + 1)), 0, stream, src, numel, (uint32_t)p.group, p.rows,
                         weights, scales);
    } else {
      const bool fills = p.group % TILE_ELEMS == 0, half_idle = p.group < 6 * TILE_ELEMS / 5;
      const bool past = streamed && p.group <= 4096 && !(fills && SR) && !(half_idle && INT4_F32);
      const bool per_lane = fills || (INT4_F32 && (p.group <= 3 * TILE_ELEMS || bytes < 40000000));
      const auto wide = past       ? eco_quantize_wide_kernel<FMT, SC, SR, false, STREAM_GROUP>
                        : per_lane ? eco_quantize_wide_kernel<FMT, SC, SR, false, PER_LANE>
                                   : eco_quantize_wide_kernel<FMT, SC, SR, false, CACHED>;
      ECO_LAUNCH_CHECKED(wide, dim3((unsigned)((numel + p.group - 1) / p.group)), dim3((unsigned)((p.group + TILE_ELEMS - 1) / TILE_ELEMS) * 64), 0,
                         stream, src, numel, (uint32_t)p.group, 1u, weights, scales);
    }
  } else if (numel <= MAX_WIDE_GROUP) {
    // one scale for a tensor that one workgroup holds: one group (4001 elements, us: in two passes, with their event, 8.9, so 4.3)
    if (numel <= static_cast<uint64_t>(TILE_ELEMS))
      ECO_LAUNCH_CHECKED(row, dim3(1), dim3(WG_THREADS), 0, stream, src, numel, (uint32_t)numel, 1u, weights, scales);
    else
      ECO_LAUNCH_CHECKED((eco_quantize_wide_kernel<FMT, SC, SR, false, CACHED>), dim3(1), dim3((unsigned)tiles * 64), 0, stream, src, numel,
                         (uint32_t)numel, 1u, weights, scales);
  } else {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= QuantSlotRing::MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_quant_ring.mu);
    const uint32_t slot = g_quant_ring.next[dev]++ % QUANT_SLOTS;
    hipEvent_t &done = g_quant_ring.done[dev][slot];
    if (done) {
      e = hipStreamWaitEvent(stream, done, 0);          // the slot's previous user, on whatever stream it ran
      if (e != hipSuccess) return e;
    } else {
      e = hipEventCreateWithFlags(&done, hipEventDisableTiming);
      if (e != hipSuccess) { done = nullptr; return e; }
    }
    constexpr uint64_t max_share = (uint64_t)QUANT_MAX_THREADS * ELEMS_PER_LANE;
    const uint64_t want = (numel + max_share - 1) / max_share;
    const uint32_t parts = want < QUANT_PARTS ? (uint32_t)want : QUANT_PARTS;
    const bool past = src_bytes >= STREAM_BYTES;
    const auto maximum = past ? eco_quantize_max_kernel<SR, STREAM_GROUP> : eco_quantize_max_kernel<SR, CACHED>;
    const auto second = past ? eco_quantize_tensorwise_kernel<FMT, SC, SR, STREAM_GROUP> : eco_quantize_tensorwise_kernel<FMT, SC, SR, PER_LANE>;
    ECO_LAUNCH_CHECKED(maximum, dim3(parts), dim3(QUANT_MAX_THREADS), 0, stream, src, numel, slot, parts);
    ECO_FLAT_CHECKED(flat_launch(numel, QUANT_PARTS), QUANT_PARTS, stream, second, src, numel,
                     parts, weights, scales, slot);
    e = hipEventRecord(done, stream);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_quantize_init(const void *src, int src_bf16, uint64_t numel, int fmt, uint64_t group_size, int scale_bf16,
                                void *weights, void *scales, hipStream_t stream) {
  const int key = (fmt == FMT_INT4 ? 4 : 0) | (scale_bf16 ? 2 : 0) | (src_bf16 ? 1 : 0);
  switch (key) {
    case 0: return launch_quantize_t<FMT_FP8, false, false>(src, numel, group_size, weights, scales, stream);
    case 1: return launch_quantize_t<FMT_FP8, false, true>(src, numel, group_size, weights, scales, stream);
    case 2: return launch_quantize_t<FMT_FP8, true, false>(src, numel, group_size, weights, scales, stream);
    case 3: return launch_quantize_t<FMT_FP8, true, true>(src, numel, group_size, weights, scales, stream);
    case 4: return launch_quantize_t<FMT_INT4, false, false>(src, numel, group_size, weights, scales, stream);
    case 5: return launch_quantize_t<FMT_INT4, false, true>(src, numel, group_size, weights, scales, stream);
    case 6: return launch_quantize_t<FMT_INT4, true, false>(src, numel, group_size, weights, scales, stream);
    default: return launch_quantize_t<FMT_INT4, true, true>(src, numel, group_size, weights, scales, stream);
  }
}

// ------------------------------------------------------------------------ dequantizer, quantization error
// SRC == 0: dst[i] = dec(code_i) * scale[i / group_size] (Sec. 3.1, x^ = s*y).
// SRC == 1 / 2: dst[i] = src[i] - dec(code_i) * scale[i / group_size] for an fp32 / bf16 source: the
// quantization error e = theta - q(theta) of the notation paragraph of Sec. 3.1 (one multiplication, one
// subtraction, each rounded to fp32).
// A lane's 8 elements may straddle two groups when the group size is not a multiple of 8, so the scale
// index is then taken per element.
// The group of a lane: a shift where the group size is a power of two, else a product with its reciprocal in double
// precision (exact to within one for the 2^35 elements of a call, then corrected); a 64-bit division is ~150 instructions
// and made the kernel arithmetic bound.
struct GroupOf { uint64_t size; double reciprocal; int32_t shift; };       // shift < 0: no power of two
// With a source, workgroups of one wave that load it behind the scale; for long arrays workgroups of two waves with every
// load of a lane under way together.  Measured, us, one wave / two -- bf16 source, INT4: 5 M elements 6.6 / 6.8, 10 M 11.1 /
// 12.9, 100 M 109 / 114, 450 M 486 / 481 (FP8 528 / 512); fp32 source, INT4: 5 M 6.9 / 7.7, 10 M 13.6 / 14.5, 20 M 27.2 /
// 26.5, 40 M 60.2 / 58.9, 200 M 292 / 284.  (The threads are a template parameter: a kernel that asks for blockDim is passed
// 256 bytes of arguments more, 0.8 us of a call.)
// Stores of fp32 cover whole lines (see exchange_chunks: INT4, 2.9 M elements 4.9 -> 4.3 us, FP8 12 M in groups of 1000 11.3 -> 10.2), and from
// 280 MB of arrays on they and the loads go past the caches.  us, before / so, usual: FP8 70 M 61.4 / 50.8, 59.4, INT4 70 M 62.4 / 54.5, 62.8, 200 M
// 167 / 155, 170 (below, 225 MB: 34.3 / 41.1, 34.4); with a source FP8 from fp32 35 M 54.1 / 50.6, 51.8, 150 M 229 / 209, 228, INT4 from bf16
// 60 M 68.0 / 60.6, 65.3, 200 M 215 / 199, 214.  Without the hint on the stores (STREAM_GROUP) errors of up to 700 MB alone take 8 % less, but they
// push the source out of the cache before HBM: with the quantizer before them 60 M from bf16 119 instead of 103.
inline bool long_error_call(int src_kind, uint64_t numel) { return numel >= (src_kind == 1 ? 1ull << 24 : 1ull << 28); }

template <int FMT, bool SCALE_BF16, int SRC, int THREADS, int ACC, int CP>
__device__ __forceinline__ void dequantize_lane(const void *weights, const void *scales, uint64_t first, int nvalid, const GroupOf &group,
                                                const void *src, float *dst) {
  const WavePieces wp = ACC == ACC_FULL ? full_wave(first) : wave_pieces(first, nvalid);
  uint32_t c[2] = {0, 0};
  if (wp.any_whole) load_codes8<FMT, ACC_FULL, CP>(weights, wp.from, 8, c);
  if (wp.any_cut) {
    if (nvalid & 7) load_ragged_codes8<FMT>(weights, first, nvalid, c);
  }
  float t[8];
  if (SRC != 0 && THREADS == 128) load_wave<SRC == 2, ACC, CP>(src, first, nvalid, wp, t);
  const uint64_t e0 = ACC == ACC_FULL || nvalid > 0 ? first : 0;          // lanes beyond the end read the first scale
  uint64_t sg;
  if (group.shift >= 0) {
    sg = e0 >> group.shift;
  } else {
    sg = (uint64_t)((double)e0 * group.reciprocal);
    const int64_t rest = (int64_t)(e0 - sg * group.size);
    if (rest < 0) --sg;
    else if (rest >= (int64_t)group.size) ++sg;
  }
  const float s0 = load_scale<SCALE_BF16>(scales, sg);
  float x[8];
  x[0] = decode_elem<FMT, 0>(c); x[1] = decode_elem<FMT, 1>(c); x[2] = decode_elem<FMT, 2>(c); x[3] = decode_elem<FMT, 3>(c);
  x[4] = decode_elem<FMT, 4>(c); x[5] = decode_elem<FMT, 5>(c); x[6] = decode_elem<FMT, 6>(c); x[7] = decode_elem<FMT, 7>(c);
  if (group.size % ELEMS_PER_LANE == 0) {
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] *= s0;
  } else {                                                  // the next group may start within the lane
    const uint64_t boundary = (sg + 1) * group.size - e0;
    const float s1 = boundary < (uint64_t)nvalid ? load_scale<SCALE_BF16>(scales, sg + 1) : s0;
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] *= ((uint64_t)j < boundary ? s0 : s1);
  }
  if (SRC != 0) {
    if (THREADS != 128) load_wave<SRC == 2, ACC, CP>(src, first, nvalid, wp, t);
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = t[j] - x[j];
  }
  store_wave8<false, ACC, CP>(dst, first, nvalid, wp, x);
}

template <int FMT, bool SCALE_BF16, int SRC, int THREADS, int CP>
__global__ __launch_bounds__(THREADS) void eco_dequantize_kernel(const void *weights, const void *scales, uint64_t numel,
                                                                         GroupOf group, const void *src, float *dst, uint32_t first_wg) {
  const uint64_t first = ((uint64_t)first_wg + blockIdx.x) * (THREADS * ELEMS_PER_LANE), e0 = first + threadIdx.x * ELEMS_PER_LANE;
  if (first + THREADS * ELEMS_PER_LANE <= numel)
    dequantize_lane<FMT, SCALE_BF16, SRC, THREADS, ACC_FULL, CP>(weights, scales, e0, 8, group, src, dst);
  else
    dequantize_lane<FMT, SCALE_BF16, SRC, THREADS, ACC_LANE, CP>(weights, scales, e0, valid_from(e0, numel), group, src, dst);
}

// src_kind: 0 = no source (plain de-quantization), 1 = fp32 source, 2 = bf16 source (dst = src - q)
hipError_t launch_dequantize(const void *weights, const void *scales, uint64_t numel, int fmt, uint64_t group_size,
                             int scale_bf16, const void *src, int src_kind, float *dst, hipStream_t stream) {
  const bool longer = long_error_call(src_kind, numel);
  // a group that holds the whole tensor: any power of two beyond it does, and no lane crosses its end
  GroupOf group = {group_size, 1.0 / (double)group_size, log2_exact(group_size)};
  if (group_size >= numel) group = {1ull << 62, 0.0, 62};
  const bool streamed = numel * (src_kind == 0 ? 4 : src_kind == 1 ? 8 : 6) + (fmt == FMT_INT4 ? numel / 2 : numel) >= STREAM_BYTES;
#define ECO_LAUNCH(F, SC, SK, T)                                                                                                              \
  do {                                                                                                                                        \
    if (streamed) ECO_FLAT_CHECKED(flat_launch(numel, T), T, stream, (eco_dequantize_kernel<F, SC, SK, T, (SK == 0 ? STREAM_GROUP : STREAM_WAVE)>), weights, scales, numel, group, src, dst); \
    else ECO_FLAT_CHECKED(flat_launch(numel, T), T, stream, (eco_dequantize_kernel<F, SC, SK, T, CACHED>), weights, scales, numel, group, src, dst); \
  } while (0)
#define ECO_LAUNCH_SRC(F, SC)                                        \
  do {                                                               \
    if (src_kind == 0) ECO_LAUNCH(F, SC, 0, 64);                     \
    else if (src_kind == 1 && longer) ECO_LAUNCH(F, SC, 1, 128);     \
    else if (src_kind == 1) ECO_LAUNCH(F, SC, 1, 64);                \
    else if (longer) ECO_LAUNCH(F, SC, 2, 128);                      \
    else ECO_LAUNCH(F, SC, 2, 64);                                   \
  } while (0)
  if (fmt == FMT_FP8) { if (scale_bf16) ECO_LAUNCH_SRC(FMT_FP8, true); else ECO_LAUNCH_SRC(FMT_FP8, false); }
  else { if (scale_bf16) ECO_LAUNCH_SRC(FMT_INT4, true); else ECO_LAUNCH_SRC(FMT_INT4, false); }
#undef ECO_LAUNCH_SRC
#undef ECO_LAUNCH
  return hipSuccess;
}

// ------------------------------------------------------------------------ bandwidth probes
// Measurement aids: what the memory system delivers for the step's own access pattern with the arithmetic
// taken out.  MIX: every lane loads what a lane of the FP8 / fp32-state Adam step loads for its 8 elements
// (8 B codes, 16 B gradient, 2 x 16 B m, 2 x 16 B v, the block's scale) and stores what it stores (codes, m, v,
// scale), in the same tile geometry, whole lines to an instruction, past the caches where the step passes them by, and under the same
// occupancy cap: 11.03 bytes read and 9.03 written per element.  COPY: the plain two-stream copy, 16 B per lane and instruction (4 B read, 4 B
// written per element).  In 32 bytes to a lane and through the caches, as the step once went, MIX was no ceiling of it: GB/s, so / now, 40 M
// elements 5298 / 6497, 1 G 5587 / 6751, 5 G 5334 / 6532; COPY through the caches / past them 6040 / 6630, 6239 / 6698, 6241 / 6708.
template <int CP>
__global__ __launch_bounds__(WG_THREADS, 8) void eco_probe_mix_kernel(void *codes, float *scales, const void *grad, void *m, void *v) {
  const uint64_t i = (uint64_t)blockIdx.x * WG_THREADS + threadIdx.x, e0 = i * ELEMS_PER_LANE;        // the lane's 8-element piece
  const WavePieces wp = full_wave(e0);
  __builtin_amdgcn_s_setprio(3);
  eco_u32x4_t g[2], mq[2], vq[2];
  uint32_t c[2];
  load_wave8<true, true, CP>(grad, wp, g);
  load_wave8<false, true, CP>(m, wp, mq);
  load_wave8<false, true, CP>(v, wp, vq);
  load_codes8<FMT_FP8, ACC_FULL, CP>(codes, e0, 8, c);
  const float s = scales[i >> 4];
  __builtin_amdgcn_s_setprio(0);
  // every loaded value reaches a store, so that no load can be dropped
  c[0] ^= g[0].x ^ g[0].z;
  c[1] ^= g[0].y ^ g[0].w;
  float mx[8], vx[8];
  unpack8<false>(mq, mx);
  unpack8<false>(vq, vx);
  mx[0] += s * 0.0f;
  store_wave_codes8<FMT_FP8, ACC_FULL, CP>(codes, e0, 8, wp, c);
  store_wave8<false, ACC_FULL, CP>(m, e0, 8, wp, vx);
  store_wave8<false, ACC_FULL, CP>(v, e0, 8, wp, mx);
  if ((threadIdx.x & 15) == 0) scales[i >> 4] = s;
}

template <int CP>
__global__ __launch_bounds__(256) void eco_probe_copy_kernel(const eco_u32x4_t *src, void *dst) {
  const eco_u32x4_t x = load_vec<CP>(src + (uint64_t)blockIdx.x * 256 + threadIdx.x);
  __builtin_amdgcn_raw_buffer_store_b128(x, buffer_at(dst, (uint64_t)blockIdx.x * 4096, 4096), threadIdx.x * 16, 0, CP);
}

hipError_t launch_bandwidth_probe(int kind, void *codes, void *scales, const void *grad, void *m, void *v, uint64_t numel, bool streamed,
                                  uint32_t lds_bytes, hipStream_t stream) {
  if (kind == 0) {
    const auto kernel = streamed ? eco_probe_mix_kernel<STREAM_WAVE> : eco_probe_mix_kernel<CACHED>;
    ECO_LAUNCH_CHECKED(kernel, dim3((unsigned)(numel / TILE_ELEMS)), dim3(WG_THREADS), lds_bytes, stream, codes, static_cast<float *>(scales), grad,
                       m, v);
  } else {
    const auto kernel = streamed ? eco_probe_copy_kernel<STREAM_WAVE> : eco_probe_copy_kernel<CACHED>;
    ECO_LAUNCH_CHECKED(kernel, dim3((unsigned)(numel / 1024)), dim3(256), 0, stream, static_cast<const eco_u32x4_t *>(m), v);
  }
  return hipSuccess;
}

// ------------------------------------------------------------------------ arithmetic self-test
// The step kernels replace sqrtf() and `/` by shorter sequences inside stated operand ranges; these kernels
// compare the short forms with the long ones for every fp32 bit pattern of [bits_lo, bits_hi) and count the
// patterns on which they differ (expected: none).
template <int KIND>
__global__ __launch_bounds__(256) void eco_selftest_kernel(float numerator, uint32_t bits_lo, uint32_t bits_hi,
                                                           unsigned long long *mismatches) {
  const uint64_t n = (uint64_t)bits_hi - bits_lo;
  unsigned bad = 0;
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (uint64_t)gridDim.x * 256) {
    const float x = u2f(bits_lo + (uint32_t)i);
    float fast, ref;
    if (KIND == 0) { fast = sqrt_rn_midrange(x); ref = sqrtf(x); }
    else { fast = div_rn_midrange(numerator, x); ref = numerator / x; }
    bad += f2u(fast) != f2u(ref);
  }
  if (bad) atomicAdd(mismatches, (unsigned long long)bad);
}

hipError_t launch_arith_selftest(int kind, float numerator, uint32_t bits_lo, uint32_t bits_hi, unsigned long long *mismatches,
                                 hipStream_t stream) {
  if (kind == 0)
    ECO_LAUNCH_CHECKED(eco_selftest_kernel<0>, dim3(256 * 16), dim3(256), 0, stream, numerator, bits_lo, bits_hi, mismatches);
  else
    ECO_LAUNCH_CHECKED(eco_selftest_kernel<1>, dim3(256 * 16), dim3(256), 0, stream, numerator, bits_lo, bits_hi, mismatches);
  return hipSuccess;
}

// ------------------------------------------------------------------------ raw Philox stream
__global__ __launch_bounds__(WG_THREADS) void eco_philox_kernel(uint32_t seed_lo, uint32_t seed_hi, uint32_t step_lo,
                                                                uint32_t tensor_id, uint64_t first_word,
                                                                uint64_t n_words, uint32_t *dst) {
  // thread t produces call (first_word >> 2) + t and writes those of its four words that are in range
  const uint64_t first_call = first_word >> 2;
  const uint64_t last_word = first_word + n_words;   // exclusive
  const uint64_t ncalls = ((last_word + 3) >> 2) - first_call;
  for (uint64_t t = (uint64_t)blockIdx.x * WG_THREADS + threadIdx.x; t < ncalls; t += (uint64_t)gridDim.x * WG_THREADS) {
    const uint64_t q = first_call + t;
    const Philox4 r = philox4x32_10((uint32_t)q, (uint32_t)(q >> 32), step_lo, tensor_id, seed_lo, seed_hi);
    const uint32_t w[4] = {r.w0, r.w1, r.w2, r.w3};
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const uint64_t j = q * 4 + k;
      if (j >= first_word && j < last_word) dst[j - first_word] = w[k];
    }
  }
}

hipError_t launch_philox_fill(uint64_t seed, uint64_t step, uint32_t tensor_id, uint64_t first_word, uint64_t n_words,
                              uint32_t *dst, hipStream_t stream) {
  const uint64_t ncalls = ((first_word + n_words + 3) >> 2) - (first_word >> 2);
  uint64_t grid = (ncalls + WG_THREADS - 1) / WG_THREADS;
  if (grid > 65536) grid = 65536;
  if (grid == 0) grid = 1;
  hipLaunchKernelGGL(eco_philox_kernel, dim3((unsigned)grid), dim3(WG_THREADS), 0, stream, (uint32_t)seed,
                     (uint32_t)(seed >> 32), (uint32_t)step, tensor_id, first_word, n_words, dst);
  return hipGetLastError();
}

}  // namespace eco
