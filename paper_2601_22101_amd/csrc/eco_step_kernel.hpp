// The fused ECO step kernel for quantized tensors (FP8-E4M3 or INT4 codes with per-block scales).
//
// One pass over memory per step: every lane owns 8 consecutive elements, loads their codes,
// gradient and optimizer state, de-quantizes, applies the optimizer update (Alg. 1 line 1 with
// the Adam form of Sec. 3.2, or the SGDM recurrences of Sec. 3.3.1), reduces the block's abs-max
// across the B/8 lanes that share a scale (Sec. 3.1, s = max|x|/rho), re-quantizes with
// stochastic or nearest-even rounding, forms the quantization error and injects it into the
// first moment (Alg. 3 line 5 / Alg. 2 line 5), and stores codes, scale, m and v.
//
// The arithmetic is a fixed sequence of single IEEE fp32 operations (the build disables
// contraction; fused multiply-adds are explicit), so that the codes and scales it produces can
// be reproduced bit for bit elsewhere:
//   w  = dec(code) * s_old            g = f32(bf16 gradient)
//   m~ = fma(b1, m, omb1*g)           v~ = fma(b2, v, omb2*(g*g))
//   d  = sqrt(v~ * rbc2) + eps        eta_t = c1 / d;  u = eta_t * m~   [SGDM: u = lr * m~]
//   theta~ = w - u                    [with decay: (w - wd*w) - u]
//   a = max|theta~| over the block;   s' = a / rho;  inv = rho / a
//       [bf16 scales: s' = bf16(a/rho), inv = 1/s'];  if inv is not finite: s' = inv = 0
//   y = theta~ * inv;  code' = round(y);  q = dec(code') * s';  e = theta~ - q
//   m^ = fma(kappa*d, e, m~)          [SGDM: fma(alpha, e, m~)]
// Variants (template parameter ALGO):
//   exact injection (Appendix A, SGDM):  m^ = fma(-inv_lr_beta, e, fma(inv_lr, e_old, m~)), e stored for the next step
//   master weights (Sec. 3.1):           w is read from / theta~ written to an fp32 master copy, m^ = m~
#pragma once
#include "eco_device.hpp"
#include "eco_internal.hpp"

namespace eco {

template <int FMT> struct FmtTraits;
template <> struct FmtTraits<FMT_FP8> { static constexpr float RHO = 448.0f; };
template <> struct FmtTraits<FMT_INT4> { static constexpr float RHO = 7.0f; };

// ------------------------------------------------------------------ 8-element loads and stores
// Access modes of a lane's 8 consecutive elements:
//   ACC_FULL    all 8 exist in every lane: vector access, no checks (full tiles)
//   ACC_GUARDED only the first `nvalid` (possibly <= 0) exist: element-wise access in every lane; missing
//               elements read as zero and are not written (the ragged tail of a tensor)
//   ACC_LANE    decided per lane: vector access where nvalid == 8, element-wise elsewhere (wide groups,
//               whose last lanes may lie beyond the group); the step kernels load as WavePieces says
//   ACC_WHOLE   all 8 of a lane exist or none (lengths that are multiples of 8): vector access where they do
enum : int { ACC_FULL = 0, ACC_GUARDED = 1, ACC_LANE = 2, ACC_WHOLE = 3 };

template <int ACC>
__device__ __forceinline__ bool use_vector(int nvalid) {
  return ACC == ACC_FULL || ((ACC == ACC_LANE || ACC == ACC_WHOLE) && nvalid == 8);
}

typedef float eco_f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t eco_u32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t eco_u32x2_t __attribute__((ext_vector_type(2)));
// How a kernel's vector accesses treat the caches.  CACHED: as usual.  The others are for arrays that come from HBM (see stream_launches): loads
// with the non-temporal hint, and stores with the given bits of the instruction, of which sc1 writes through the L2.  Neither half alone
// helps, and neither where an instruction covers halves of lines (see exchange_chunks): a copy of the FP8 Adam step's byte mix, 268 M
// elements, us: 985; instructions over whole lines 944; with loads nt 1008, stores nt 945, both 865, loads nt and stores sc1 nt 837.
// STREAM_WAVE, of independent waves: 700 M elements in groups of 128 2390 -> 2195 (sc1 alone 2230).  STREAM_GROUP, of workgroups that store
// behind a barrier: rows of 1152 2303 -> 2118 (with nt 2473), 2304 2342 -> 2142 (2443), 3072 2384 -> 2176 (2270).
enum : int { CACHED = 0, STREAM_GROUP = 16, STREAM_WAVE = 16 | 2 };          // sc1; sc1 and nt
constexpr int POLICY_NT = 2;                       // the non-temporal hint, in a buffer instruction
template <int CP, class V>
__device__ __forceinline__ V load_vec(const V *p) { return CP != CACHED ? __builtin_nontemporal_load(p) : *p; }

template <int ACC>
__device__ __forceinline__ void load_f32x8(const float *p, int nvalid, float (&out)[8]) {
  if (use_vector<ACC>(nvalid)) {
    const float4 a = reinterpret_cast<const float4 *>(p)[0];
    const float4 b = reinterpret_cast<const float4 *>(p)[1];
    out[0] = a.x; out[1] = a.y; out[2] = a.z; out[3] = a.w;
    out[4] = b.x; out[5] = b.y; out[6] = b.z; out[7] = b.w;
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) out[j] = ACC != ACC_WHOLE && j < nvalid ? p[j] : 0.0f;
  }
}

template <int ACC>
__device__ __forceinline__ void load_bf16x8(const uint16_t *p, int nvalid, float (&out)[8]) {
  if (use_vector<ACC>(nvalid)) {
    const eco_u32x4_t q = *reinterpret_cast<const eco_u32x4_t *>(p);
    out[0] = bf16_lo(q.x); out[1] = bf16_hi(q.x); out[2] = bf16_lo(q.y); out[3] = bf16_hi(q.y);
    out[4] = bf16_lo(q.z); out[5] = bf16_hi(q.z); out[6] = bf16_lo(q.w); out[7] = bf16_hi(q.w);
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) out[j] = ACC != ACC_WHOLE && j < nvalid ? u2f((uint32_t)p[j] << 16) : 0.0f;
  }
}

template <int ACC>
__device__ __forceinline__ void store_f32x8(float *p, int nvalid, const float (&x)[8]) {
  if (use_vector<ACC>(nvalid)) {
    reinterpret_cast<eco_f32x4_t *>(p)[0] = eco_f32x4_t{x[0], x[1], x[2], x[3]};
    reinterpret_cast<eco_f32x4_t *>(p)[1] = eco_f32x4_t{x[4], x[5], x[6], x[7]};
  } else if (ACC != ACC_WHOLE) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (j < nvalid) p[j] = x[j];
  }
}

template <int ACC>
__device__ __forceinline__ void store_bf16x8(uint16_t *p, int nvalid, const float (&x)[8]) {
  uint32_t h[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) h[j] = f32x2_to_bf16x2_rne(x[2 * j], x[2 * j + 1]);
  if (use_vector<ACC>(nvalid)) {
    *reinterpret_cast<eco_u32x4_t *>(p) = eco_u32x4_t{h[0], h[1], h[2], h[3]};
  } else if (ACC != ACC_WHOLE) {
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (j < nvalid) p[j] = (uint16_t)(h[j >> 1] >> (16 * (j & 1)));
  }
}

template <bool BF16, int ACC>
__device__ __forceinline__ void load_state8(const void *base, uint64_t e0, int nvalid, float (&out)[8]) {
  if (BF16) load_bf16x8<ACC>(static_cast<const uint16_t *>(base) + e0, nvalid, out);
  else load_f32x8<ACC>(static_cast<const float *>(base) + e0, nvalid, out);
}

// 8 codes of one lane: two dwords of E4M3 bytes, or one dword of INT4 nibbles (in c[0]).
template <int FMT, int ACC, int CP = CACHED>
__device__ __forceinline__ void load_codes8(const void *base, uint64_t e0, int nvalid, uint32_t (&c)[2]) {
  const uint8_t *p = static_cast<const uint8_t *>(base) + (FMT == FMT_FP8 ? e0 : (e0 >> 1));
  if (use_vector<ACC>(nvalid)) {
    if (FMT == FMT_FP8) {
      const eco_u32x2_t q = load_vec<CP>(reinterpret_cast<const eco_u32x2_t *>(p));
      c[0] = q.x; c[1] = q.y;
    } else {
      c[0] = load_vec<CP>(reinterpret_cast<const uint32_t *>(p)); c[1] = 0;
    }
  } else {
    c[0] = 0; c[1] = 0;
    const int nbytes = FMT == FMT_FP8 ? nvalid : (nvalid + 1) >> 1;
    constexpr int MAXB = FMT == FMT_FP8 ? 8 : 4;
#pragma unroll
    for (int k = 0; k < MAXB; ++k)
      if (ACC != ACC_WHOLE && k < nbytes) c[k >> 2] |= (uint32_t)p[k] << (8 * (k & 3));
  }
}

template <int FMT, int ACC>
__device__ __forceinline__ void store_codes8(void *base, uint64_t e0, int nvalid, const uint32_t (&c)[2]) {
  uint8_t *p = static_cast<uint8_t *>(base) + (FMT == FMT_FP8 ? e0 : (e0 >> 1));
  if (use_vector<ACC>(nvalid)) {
    if (FMT == FMT_FP8) *reinterpret_cast<eco_u32x2_t *>(p) = eco_u32x2_t{c[0], c[1]};
    else *reinterpret_cast<uint32_t *>(p) = c[0];
  } else if (ACC != ACC_WHOLE) {
    const int nbytes = FMT == FMT_FP8 ? nvalid : (nvalid + 1) >> 1;
    constexpr int MAXB = FMT == FMT_FP8 ? 8 : 4;
#pragma unroll
    for (int k = 0; k < MAXB; ++k)
      if (k < nbytes) p[k] = (uint8_t)(c[k >> 2] >> (8 * (k & 3)));
  }
}

// x_j = value for the elements of a lane that do not exist.  (ACC_LANE: seldom anything to do, so a wave-uniform branch.)
template <int ACC>
__device__ __forceinline__ void fill_missing(float (&x)[8], int nvalid, float value) {
  if (ACC == ACC_FULL || (ACC == ACC_LANE && !wave_any(nvalid < 8))) return;
#pragma unroll
  for (int j = 0; j < 8; ++j)
    if (ACC == ACC_WHOLE ? nvalid == 0 : j >= nvalid) x[j] = value;
}

// Eight fp32 elements of each lane of a wave, the lanes' pieces one behind the other: 32 bytes to a lane, which two instructions of 16
// bytes would take in halves of every 64-byte request.  So each takes 1 KB of consecutive bytes: lane l has chunk 2 l (l < 32) or
// 2 (l - 32) + 1 of the 64 and the same of the next 64, and an exchange between the halves of the wave brings a lane's two chunks
// together (four instructions; its own inverse, so stores take the same way back).
__device__ __forceinline__ uint32_t lane_chunk() { return 2 * (threadIdx.x & 31) + ((threadIdx.x >> 5) & 1); }
__device__ __forceinline__ void exchange_chunks(eco_u32x4_t (&q)[2]) {
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const auto r = __builtin_amdgcn_permlane32_swap(q[0][i], q[1][i], false, false);
    q[0][i] = r[0];
    q[1][i] = r[1];
  }
}
// The element at which the wave's first piece starts; e0: the lane's.
__device__ __forceinline__ uint64_t wave_start(uint64_t e0) {
  return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)e0) |
         (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(e0 >> 32)) << 32;
}
// Stores of a wave go through a buffer that ends with its last whole piece, so lanes beyond it need no branch.
typedef __amdgpu_buffer_rsrc_t buffer_t;
__device__ __forceinline__ buffer_t buffer_at(const void *base, uint64_t byte, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(static_cast<const char *>(base)) + byte, 0, (int)bytes, 0x00020000);
}
// whole: the lanes, from the first on, whose pieces exist; the others read the last of those once more, and write nothing.
template <bool FULL, int CP>
__device__ __forceinline__ void load_f32_wave(const void *base, uint64_t wave, int whole, eco_u32x4_t (&q)[2]) {
  const char *p = static_cast<const char *>(base) + wave * 4;
  const uint32_t c = lane_chunk(), last = 2 * (uint32_t)whole - 2 + (c & 1), c0 = FULL || c < last ? c : last, c1 = FULL || c + 64 < last ? c + 64 : last;
  q[0] = load_vec<CP>(reinterpret_cast<const eco_u32x4_t *>(p + c0 * 16));
  q[1] = load_vec<CP>(reinterpret_cast<const eco_u32x4_t *>(p + c1 * 16));
  exchange_chunks(q);
}
__device__ __forceinline__ eco_u32x4_t pack_bf16x8(const float (&x)[8]) {
  return eco_u32x4_t{f32x2_to_bf16x2_rne(x[0], x[1]), f32x2_to_bf16x2_rne(x[2], x[3]), f32x2_to_bf16x2_rne(x[4], x[5]),
                     f32x2_to_bf16x2_rne(x[6], x[7])};
}
// The first nvalid (1..7) elements of a piece, zeros behind them.  Element by element, but without a branch, so that the loads of a
// lane are under way together: an element that does not exist is the first one read once more (25 odd tensors, SGDM, without a plan
// 7.6 -> 6.5 us, 30 of 4004 elements beside 30 plain ones 5.1 -> 4.4).
template <bool BF16>
__device__ __forceinline__ void load_ragged8(const void *base, uint64_t e, int nvalid, eco_u32x4_t (&q)[2]) {
  uint32_t x[8];
#pragma unroll
  for (int j = 0; j < 7; ++j) {
    const uint64_t i = e + (j < nvalid ? j : 0);
    x[j] = BF16 ? (uint32_t)static_cast<const uint16_t *>(base)[i] : static_cast<const uint32_t *>(base)[i];
  }
  x[7] = 0;
#pragma unroll
  for (int j = 1; j < 7; ++j) x[j] = j < nvalid ? x[j] : 0u;
  if (BF16) {
    q[0] = eco_u32x4_t{x[0] | x[1] << 16, x[2] | x[3] << 16, x[4] | x[5] << 16, x[6]};
  } else {
    q[0] = eco_u32x4_t{x[0], x[1], x[2], x[3]};
    q[1] = eco_u32x4_t{x[4], x[5], x[6], 0};
  }
}
template <int FMT>
__device__ __forceinline__ void load_ragged_codes8(const void *base, uint64_t e, int nvalid, uint32_t (&c)[2]) {
  constexpr int MAXB = FMT == FMT_FP8 ? 7 : 4;
  const uint8_t *p = static_cast<const uint8_t *>(base) + (FMT == FMT_FP8 ? e : e >> 1);
  const int nbytes = FMT == FMT_FP8 ? nvalid : (nvalid + 1) >> 1;
  uint32_t x[8] = {};
#pragma unroll
  for (int k = 0; k < MAXB; ++k) x[k] = p[k < nbytes ? k : 0];
#pragma unroll
  for (int k = 1; k < MAXB; ++k) x[k] = k < nbytes ? x[k] : 0u;
  c[0] = x[0] | x[1] << 8 | x[2] << 16 | x[3] << 24;
  c[1] = x[4] | x[5] << 8 | x[6] << 16;
}
template <bool BF16>
__device__ __forceinline__ void unpack8(const eco_u32x4_t (&q)[2], float (&x)[8]) {
  if (BF16) {
    x[0] = bf16_lo(q[0].x); x[1] = bf16_hi(q[0].x); x[2] = bf16_lo(q[0].y); x[3] = bf16_hi(q[0].y);
    x[4] = bf16_lo(q[0].z); x[5] = bf16_hi(q[0].z); x[6] = bf16_lo(q[0].w); x[7] = bf16_hi(q[0].w);
  } else {
    x[0] = u2f(q[0].x); x[1] = u2f(q[0].y); x[2] = u2f(q[0].z); x[3] = u2f(q[0].w);
    x[4] = u2f(q[1].x); x[5] = u2f(q[1].y); x[6] = u2f(q[1].z); x[7] = u2f(q[1].w);
  }
}

// What a wave whose last lanes may lie beyond the end reads (ACC_LANE; its lanes' pieces of 8 elements are consecutive).  A
// load inside a branch of its own is waited for there, one array after the other, which is what bounded such waves.  So all
// loads of all lanes are vectors and issued together: a lane beyond the end reads the wave's last whole piece once more (no
// traffic, and nothing that a maximum would notice, as long as no piece is cut off: a cut one may begin a group, whose other lanes then
// hold another group's elements and have to be cleared, see `fill`), and writes nothing.  Only the one lane whose piece is cut off reads
// element by element, over what it has been given, in a branch that waves without one skip.  Measured (us, five loads waited for in
// turn / this): Adam, fp32 state, 44 tensors of 1001 rows of 2304 538 / 403, 30 750 rows of 1152 in INT4 180 / 133.
struct WavePieces {
  bool any_whole, any_cut;       // wave-uniform
  int last;                      // the lane with the last whole piece
  uint64_t from;                 // where the lane reads its vectors
  int fill;                      // how many of the lane's 8 elements stand for something
  uint64_t wave;                 // where the wave's pieces start
  int whole;                     // whole pieces
};
__device__ __forceinline__ WavePieces wave_pieces(uint64_t e0, int nvalid) {
  const int lane = (int)(threadIdx.x & 63);
  const uint64_t whole = __builtin_amdgcn_ballot_w64(nvalid == 8);
  WavePieces p;
  p.any_whole = whole != 0;
  p.any_cut = wave_any((nvalid & 7) != 0);
  p.last = 63 - __builtin_clzll(whole | 1);
  p.from = e0 - (uint64_t)(lane > p.last ? lane - p.last : 0) * ELEMS_PER_LANE;
  p.fill = p.any_cut || !p.any_whole ? nvalid : 8;
  p.wave = wave_start(e0);
  p.whole = p.any_whole ? p.last + 1 : 0;
  return p;
}
__device__ __forceinline__ WavePieces full_wave(uint64_t e0) { return WavePieces{true, false, 63, e0, 8, wave_start(e0), 64}; }

// Optimizer state, master weights (fp32) or the stored error of the wave's lanes.
template <bool BF16, bool FULL, int CP>
__device__ __forceinline__ void load_wave8(const void *base, const WavePieces &wp, eco_u32x4_t (&q)[2]) {
  if (BF16) q[0] = load_vec<CP>(reinterpret_cast<const eco_u32x4_t *>(static_cast<const uint16_t *>(base) + wp.from));
  else load_f32_wave<FULL, CP>(base, wp.wave, wp.whole, q);
}
template <bool BF16, int ACC, int CP>
__device__ __forceinline__ void store_wave8(void *base, uint64_t e0, int nvalid, const WavePieces &wp, const float (&x)[8]) {
  if (ACC != ACC_FULL && ACC != ACC_LANE) {
    if (BF16) store_bf16x8<ACC>(static_cast<uint16_t *>(base) + e0, nvalid, x);
    else store_f32x8<ACC>(static_cast<float *>(base) + e0, nvalid, x);
    return;
  }
  constexpr uint32_t ES = BF16 ? 2 : 4;
  const buffer_t b = buffer_at(base, wp.wave * ES, (uint32_t)wp.whole * (8 * ES));
  if (BF16) {
    __builtin_amdgcn_raw_buffer_store_b128(pack_bf16x8(x), b, (threadIdx.x & 63) * 16, 0, CP);
  } else {
    eco_u32x4_t q[2] = {{f2u(x[0]), f2u(x[1]), f2u(x[2]), f2u(x[3])}, {f2u(x[4]), f2u(x[5]), f2u(x[6]), f2u(x[7])}};
    exchange_chunks(q);
    __builtin_amdgcn_raw_buffer_store_b128(q[0], b, lane_chunk() * 16, 0, CP);
    __builtin_amdgcn_raw_buffer_store_b128(q[1], b, lane_chunk() * 16 + 1024, 0, CP);
  }
  if (ACC == ACC_LANE && wp.any_cut && nvalid < 8) {
    if (BF16) store_bf16x8<ACC_GUARDED>(static_cast<uint16_t *>(base) + e0, nvalid, x);
    else store_f32x8<ACC_GUARDED>(static_cast<float *>(base) + e0, nvalid, x);
  }
}
template <int FMT, int ACC, int CP>
__device__ __forceinline__ void store_wave_codes8(void *base, uint64_t e0, int nvalid, const WavePieces &wp, const uint32_t (&c)[2]) {
  if (ACC != ACC_FULL && ACC != ACC_LANE) {
    store_codes8<FMT, ACC>(base, e0, nvalid, c);
    return;
  }
  if (FMT == FMT_FP8)
    __builtin_amdgcn_raw_buffer_store_b64(eco_u32x2_t{c[0], c[1]}, buffer_at(base, wp.wave, (uint32_t)wp.whole * 8), (threadIdx.x & 63) * 8, 0,
                                          CP);
  else
    __builtin_amdgcn_raw_buffer_store_b32(c[0], buffer_at(base, wp.wave >> 1, (uint32_t)wp.whole * 4), (threadIdx.x & 63) * 4, 0, CP);
  if (ACC == ACC_LANE && wp.any_cut && nvalid < 8) store_codes8<FMT, ACC_GUARDED>(base, e0, nvalid, c);
}

template <int FMT, int J>
__device__ __forceinline__ float decode_elem(const uint32_t (&c)[2]) {
  if (FMT == FMT_FP8) return e4m3_decode<(J & 3)>(c[J >> 2]);
  return int4_decode_sixteenth<J>(c[0], c[0] >> 4) * 16.0f;
}

// The decoded values dq_j of a lane's 8 codes and the factor sc with w_j = dq_j * sc (INT4 decodes to
// sixteenths, so sc = 16 s there: exact, see int4_decode_sixteenth).
template <int FMT>
__device__ __forceinline__ float decode8(const uint32_t (&c)[2], float s, float (&dq)[8]) {
  if (FMT == FMT_FP8) {
    dq[0] = e4m3_decode<0>(c[0]); dq[1] = e4m3_decode<1>(c[0]); dq[2] = e4m3_decode<2>(c[0]); dq[3] = e4m3_decode<3>(c[0]);
    dq[4] = e4m3_decode<0>(c[1]); dq[5] = e4m3_decode<1>(c[1]); dq[6] = e4m3_decode<2>(c[1]); dq[7] = e4m3_decode<3>(c[1]);
    return s;
  }
  uint32_t hi = c[0] >> 4;
  asm volatile("" : "+v"(hi));          // keep the shifted copy in a register: each nibble is then one byte-select away
  dq[0] = int4_decode_sixteenth<0>(c[0], hi); dq[1] = int4_decode_sixteenth<1>(c[0], hi);
  dq[2] = int4_decode_sixteenth<2>(c[0], hi); dq[3] = int4_decode_sixteenth<3>(c[0], hi);
  dq[4] = int4_decode_sixteenth<4>(c[0], hi); dq[5] = int4_decode_sixteenth<5>(c[0], hi);
  dq[6] = int4_decode_sixteenth<6>(c[0], hi); dq[7] = int4_decode_sixteenth<7>(c[0], hi);
  return s * 16.0f;
}

template <bool BF16>
__device__ __forceinline__ float load_scale(const void *scales, uint64_t blk) {
  if (BF16) return u2f((uint32_t)static_cast<const uint16_t *>(scales)[blk] << 16);
  return static_cast<const float *>(scales)[blk];
}

// abs-max scale of a block from a = max|x| (identical in all lanes of the block)
template <int FMT, bool SCALE_BF16>
__device__ __forceinline__ void block_scale(float a, float &s_new, float &inv) {
  constexpr float RHO = FmtTraits<FMT>::RHO;
  s_new = a / RHO;
  if (SCALE_BF16) {
    s_new = u2f(f32_to_bf16_rne(s_new) << 16);
    inv = 1.0f / s_new;
  } else {
    inv = RHO / a;
  }
  if (!(inv < __builtin_inff())) { s_new = 0.0f; inv = 0.0f; }   // a == 0, or rho/a overflows
}

__device__ __forceinline__ float absmax8(const float (&x)[8]) {
  float a = __builtin_fmaxf(__builtin_fabsf(x[0]), __builtin_fabsf(x[1]));
#pragma unroll
  for (int j = 2; j < 8; ++j) a = __builtin_fmaxf(a, __builtin_fabsf(x[j]));
  return a;
}

__device__ __forceinline__ float absmin8(const float (&x)[8]) {
  float a = __builtin_fminf(__builtin_fabsf(x[0]), __builtin_fabsf(x[1]));
#pragma unroll
  for (int j = 2; j < 8; ++j) a = __builtin_fminf(a, __builtin_fabsf(x[j]));
  return a;
}

// Encode y_j = x_j * inv (j = 0..7) onto the grid: packed codes in c, and in q the values the new codes decode
// to (before scaling).  r = the lane's Philox words.
template <int FMT, int ROUND, bool NORMAL_ONLY>
__device__ __forceinline__ void encode8(const float (&x)[8], float inv, const Philox4 &r, uint32_t (&c)[2], float (&q)[8]) {
  const uint32_t rw[4] = {r.w0, r.w1, r.w2, r.w3};
  c[1] = 0;
  if (FMT == FMT_FP8) {
    // inv >= 0, so the sign of y is the sign of x
    uint32_t t[8];
#define ECO_FP8_ELEM(J) t[J] = e4m3_encode_top<ROUND, NORMAL_ONLY, (J & 1)>(__builtin_fabsf(x[J]) * inv, rw[J >> 1], f2u(x[J]));
    ECO_FP8_ELEM(0) ECO_FP8_ELEM(1) ECO_FP8_ELEM(2) ECO_FP8_ELEM(3)
    ECO_FP8_ELEM(4) ECO_FP8_ELEM(5) ECO_FP8_ELEM(6) ECO_FP8_ELEM(7)
#undef ECO_FP8_ELEM
    c[0] = pack_top_bytes4(t[0], t[1], t[2], t[3]);
    c[1] = pack_top_bytes4(t[4], t[5], t[6], t[7]);
    q[0] = e4m3_decode<0>(c[0]); q[1] = e4m3_decode<1>(c[0]); q[2] = e4m3_decode<2>(c[0]); q[3] = e4m3_decode<3>(c[0]);
    q[4] = e4m3_decode<0>(c[1]); q[5] = e4m3_decode<1>(c[1]); q[6] = e4m3_decode<2>(c[1]); q[7] = e4m3_decode<3>(c[1]);
  } else {
    uint32_t even = 0, odd = 0;
#define ECO_INT4_ELEM(J)                                                                              \
    q[J] = int4_round<ROUND, (J & 1)>(x[J] * inv, rw[J >> 1]);                                        \
    int4_insert<J>(q[J], even, odd);
    ECO_INT4_ELEM(0) ECO_INT4_ELEM(1) ECO_INT4_ELEM(2) ECO_INT4_ELEM(3)
    ECO_INT4_ELEM(4) ECO_INT4_ELEM(5) ECO_INT4_ELEM(6) ECO_INT4_ELEM(7)
#undef ECO_INT4_ELEM
    c[0] = int4_pack(even, odd);
  }
}

// d_j = sqrt(x_j) + eps for eight non-negative x.  When every x of the wave lies in the range of
// sqrt_rn_midrange the short sequence is used; both branches return the correctly rounded root.
// Returns whether the short sequence was used (wave-uniform): then every x of the wave lies in [2^-96, 2^96].
__device__ __forceinline__ bool sqrt_plus_eps8(const float (&x)[8], float eps, float (&d)[8]) {
  uint32_t lo = f2u(x[0]), hi = f2u(x[0]);
#pragma unroll
  for (int j = 1; j < 8; ++j) {
    const uint32_t b = f2u(x[j]);
    lo = lo < b ? lo : b;
    hi = hi > b ? hi : b;
  }
  if (wave_all(lo >= SQRT_MID_LO && hi <= SQRT_MID_HI)) {
#pragma unroll
    for (int j = 0; j < 8; ++j) d[j] = sqrt_rn_midrange(x[j]) + eps;
    return true;
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) d[j] = sqrtf(x[j]) + eps;
  return false;
}

// eta_j = c1 / d_j with d_j = sqrt(x_j) + eps: the element-wise step size of Sec. 3.2, (eta / (1 - b1^k)) / (sqrt(v^) + eps).
// After the short square root every d of the wave lies in [2^-48, 2^48 + eps], and div_mid says that eps <= 1 and c1 is
// in the range of the short division.
__device__ __forceinline__ void step_sizes8(const StepArgs &a, const float (&x)[8], float (&d)[8], float (&eta)[8]) {
  if (sqrt_plus_eps8(x, a.eps, d) && a.div_mid) {
#pragma unroll
    for (int j = 0; j < 8; ++j) eta[j] = div_rn_midrange(a.c1, d[j]);
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j) eta[j] = a.c1 / d[j];
  }
}

// ------------------------------------------------------------------ the step of one lane
// How the abs-max of a scale group is obtained:
//   RED_BLOCK  the group is 2^shift elements inside one wave: DPP/swizzle all-reduce over its lanes
//   RED_WG     the group is the whole workgroup (2..16 waves): wave all-reduce, then an LDS combine
//   RED_WG_ROWS the workgroup holds up to 16 whole groups of more than 512 elements each (a wave meets at most two of
//              them): per wave one all-reduce for each of its groups, LDS atomic max into the group's entry
//   RED_TILE   first pass of the step for a group larger than a workgroup (tensor-wise scaling): wave all-reduce, the wave's
//              maximum goes to its tile's entry of a scratch array, which a small kernel folds into the
//              tensor's slot (tens of thousands of atomics on one address serialize in the memory system)
//   RED_TILE_KEEP the same with master weights, whose new values, and the moments, are final before the scale is known: they are stored
//   RED_ROWS   groups of up to 256 elements of any length, several to a wave: segmented all-reduce over the group's lanes
//   RED_SLOT   second pass: the abs-max is read from that slot; everything is recomputed and written
//              except the scale (a last, tiny kernel writes it once every tile has used the old one)
enum : int { RED_BLOCK = 0, RED_WG = 1, RED_TILE_KEEP = 2, RED_SLOT = 3, RED_TILE = 4, RED_WG_ROWS = 5, RED_ROWS = 6 };

constexpr uint32_t WG_ROWS = 16;
// arg: RED_BLOCK: log2(group size); RED_WG_ROWS: which of the workgroup's groups the lane belongs to; RED_ROWS: the
// first lane of the lane's group.  lanes: RED_ROWS: the lanes of a group; RED_WG: the waves of the workgroup.
template <int RED>
__device__ __forceinline__ float group_absmax(float lane_max, int arg, uint32_t *slot, int lanes = 0) {
  if (RED == RED_ROWS) {
    // inclusive maximum scan within the group, doubling the distance; the group's last lane then holds its maximum
    const int lane = (int)(threadIdx.x & 63), last = arg + lanes - 1;
    uint32_t x = f2u(lane_max);
    for (int off = 1; off < lanes; off <<= 1) {                // wave-uniform
      const uint32_t o = (uint32_t)__shfl_up((int)x, off, 64);
      if (lane - off >= arg) x = x > o ? x : o;
    }
    return u2f((uint32_t)__shfl((int)x, last < 64 ? last : 63, 64));
  }
  if (RED == RED_BLOCK) return u2f(group_umax(f2u(lane_max), 1 << (arg - 3)));
  if (RED == RED_SLOT) return u2f(*slot);
  if (RED == RED_WG_ROWS) {
    __shared__ uint32_t row_max[WG_ROWS];
    if (threadIdx.x < WG_ROWS) row_max[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t x = f2u(lane_max);
    const int first = __builtin_amdgcn_readfirstlane(arg), last = __builtin_amdgcn_readlane(arg, 63);
    const uint32_t m_first = group_umax(arg == first ? x : 0u, 64);
    if ((threadIdx.x & 63) == 0) atomicMax(&row_max[first], m_first);
    if (last != first) {                                      // wave-uniform
      const uint32_t m_last = group_umax(arg == last ? x : 0u, 64);
      if ((threadIdx.x & 63) == 0) atomicMax(&row_max[last], m_last);
    }
    __syncthreads();
    return u2f(row_max[arg]);
  }
  const uint32_t wmax = group_umax(f2u(lane_max), 64);
  if (RED == RED_TILE || RED == RED_TILE_KEEP) {
    if ((threadIdx.x & 63) == 0) *slot = wmax;
    return 0.0f;
  }
  // RED_WG
  __shared__ uint32_t wave_max[16];
  const int nwaves = lanes;
  if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = wmax;
  __syncthreads();
  uint32_t r = wave_max[0];
  for (int k = 1; k < nwaves; ++k) { const uint32_t o = wave_max[k]; r = r > o ? r : o; }
  return u2f(r);
}

// A bf16 scale has 8 significant bits and a decoded code at most 4, so dec(c) * s is exact in fp32 (also where it is
// subnormal: its lowest bit is at least 2^-142) and theta~ = w - u and e = theta~ - dec(c') s' may be formed by one fused
// multiply-add each: the same real number is rounded once either way.  Until then w holds the decoded values and sc the
// factor.
template <bool SCALE_BF16, int ALGO>
constexpr bool exact_scale() { return SCALE_BF16 && !algo_is_master(ALGO); }

// m~, v~ and the argument x = v~ / (1 - b2^k) of the square root; V_FINAL: v already is v~.
template <int ALGO, bool V_FINAL = false>
__device__ __forceinline__ void moments_lane(const StepArgs &a, const float (&g)[8], float (&m)[8], float (&v)[8], float (&x)[8]) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    m[j] = fmaf(a.b1, m[j], a.omb1 * g[j]);
    if (algo_is_adam(ALGO)) {
      if (!V_FINAL) v[j] = fmaf(a.b2, v[j], a.omb2 * (g[j] * g[j]));
      x[j] = v[j] * a.rbc2;
    }
  }
}

// OPTIM_STEP on the de-quantized (or master) weights: theta~, and d for Adam.
template <bool SCALE_BF16, int ALGO, int ACC>
__device__ __forceinline__ void theta_lane(const StepArgs &a, float (&x)[8], float (&w)[8], float sc, const float (&m)[8], int nvalid,
                                           float (&d)[8], float (&th)[8]) {
  constexpr bool ADAM = algo_is_adam(ALGO), EXACT_SCALE = exact_scale<SCALE_BF16, ALGO>();
  float eta[8], u[8];
  if (ADAM) {
    fill_missing<ACC>(x, nvalid, 1.0f);                              // elements that do not exist decide nothing
    step_sizes8(a, x, d, eta);
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    if (ADAM) {
      u[j] = eta[j] * m[j];
    } else {
      d[j] = 0.0f;
      u[j] = a.lr * m[j];
    }
  }
  // decoupled decay is off in most runs, so it is kept a (wave-uniform) branch: the empty asm statements stop
  // the compiler from turning the blocks into multiply-subtract-select triples
  if (EXACT_SCALE && a.wd == 0.0f) {
    asm volatile("" ::: "memory");
#pragma unroll
    for (int j = 0; j < 8; ++j) th[j] = fmaf(w[j], sc, -u[j]);
  } else {
    if (EXACT_SCALE) {
#pragma unroll
      for (int j = 0; j < 8; ++j) w[j] *= sc;
    }
    if (a.wd != 0.0f) {
      asm volatile("" ::: "memory");
#pragma unroll
      for (int j = 0; j < 8; ++j) w[j] = w[j] - a.wd * w[j];
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) th[j] = w[j] - u[j];
  }
  fill_missing<ACC>(th, nvalid, 0.0f);
}

// The random words of a lane's 8 elements, counter e0 / 8.
template <int ROUND>
__device__ __forceinline__ Philox4 random_lane(const StepArgs &a, const TensorDesc &td, uint64_t e0, uint32_t seed_lo, uint32_t seed_hi) {
  Philox4 r = {0, 0, 0, 0};
  if (ROUND == ROUND_SR) {
    const uint64_t q = e0 >> 3;
    // tensors of up to 2^35 elements (a wave-uniform, scalar test): the high counter word is zero, so the words
    // that enter the first two rounds beside q are all wave-uniform and their products are scalar work (the
    // empty asm statement keeps the two calls apart: merged, the zero would become a per-lane select)
    if (td.numel <= (1ull << 35)) {
      r = philox4x32_10((uint32_t)q, 0u, a.step_lo, td.tensor_id, seed_lo, seed_hi);
      asm volatile("" ::: "memory");
    } else {
      r = philox4x32_10((uint32_t)q, (uint32_t)(q >> 32), a.step_lo, td.tensor_id, seed_lo, seed_hi);
    }
  }
  return r;
}

// ECO_QUANTIZE given the group's abs-max: the new codes, what they decode to and, returned, the new scale.
template <int FMT, bool SCALE_BF16, int ROUND, int ACC>
__device__ __forceinline__ float quantize_lane8(float amax, const Philox4 &r, int nvalid, const float (&th)[8], uint32_t (&cn)[2],
                                                float (&qn)[8]) {
  float s_new, inv;
  block_scale<FMT, SCALE_BF16>(amax, s_new, inv);
  if (FMT == FMT_FP8) {
    // the E4M3 subnormal range (|y| < 2^-6) needs a second formula; it is rare, so decide per wave
    // (multiplication by inv >= 0 is monotone, so the smallest |y| is fl(min|theta~| * inv))
    float lo[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) lo[j] = th[j];
    fill_missing<ACC>(lo, nvalid, __builtin_inff());
    if (wave_any(absmin8(lo) * inv < 0x1p-6f)) encode8<FMT, ROUND, false>(th, inv, r, cn, qn);
    else encode8<FMT, ROUND, true>(th, inv, r, cn, qn);
  } else {
    encode8<FMT, ROUND, true>(th, inv, r, cn, qn);
  }
  return s_new;
}

// The quantization error and its injection into m~; eo: the stored error of the exact variant, old in and new out.
template <bool SCALE_BF16, int ALGO>
__device__ __forceinline__ void inject_lane8(const StepArgs &a, float s_new, const float (&th)[8], const float (&qn)[8],
                                             const float (&d)[8], float (&m)[8], float (&eo)[8]) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const float e = SCALE_BF16 ? fmaf(-qn[j], s_new, th[j]) : th[j] - qn[j] * s_new;   // exact product, see exact_scale
    if (ALGO == ALGO_ADAM) m[j] = fmaf(a.kappa * d[j], e, m[j]);
    else if (ALGO == ALGO_SGDM) m[j] = fmaf(a.alpha, e, m[j]);
    else { m[j] = fmaf(-a.inv_lr_beta, e, fmaf(a.inv_lr, eo[j], m[j])); eo[j] = e; }
  }
}

// Both, with the stores: codes, the injected momentum (or master weights); returns the new scale.
template <int FMT, bool STATE_BF16, bool SCALE_BF16, int ALGO, int ROUND, int ACC, int CP>
__device__ __forceinline__ float quantize_inject_lane(const StepArgs &a, const TensorDesc &td, uint64_t e0, int nvalid, const WavePieces &wp,
                                                      float amax, const Philox4 &r, const float (&th)[8], const float (&d)[8],
                                                      float (&m)[8]) {
  constexpr bool MASTER = algo_is_master(ALGO);
  uint32_t cn[2];
  float qn[8];
  const float s_new = quantize_lane8<FMT, SCALE_BF16, ROUND, ACC>(amax, r, wp.fill, th, cn, qn);
  store_wave_codes8<FMT, ACC, CP>(td.w, e0, nvalid, wp, cn);
  if (MASTER) store_wave8<false, ACC, CP>(td.aux, e0, nvalid, wp, th);
  if (!MASTER) {
    float eo[8];
    if (ALGO == ALGO_SGDM_EXACT) {
      if (ACC == ACC_FULL || ACC == ACC_LANE) {
        eco_u32x4_t q[2] = {};
        if (wp.any_whole) load_wave8<false, ACC == ACC_FULL, CP>(td.aux, wp, q);
        if (wp.any_cut) {
          if (nvalid & 7) load_ragged8<false>(td.aux, e0, nvalid, q);
        }
        unpack8<false>(q, eo);
      } else {
        load_f32x8<ACC>(static_cast<const float *>(td.aux) + e0, nvalid, eo);
      }
    }
    inject_lane8<SCALE_BF16, ALGO>(a, s_new, th, qn, d, m, eo);
    if (ALGO == ALGO_SGDM_EXACT) store_wave8<false, ACC, CP>(td.aux, e0, nvalid, wp, eo);
  }
  store_wave8<STATE_BF16, ACC, CP>(td.m, e0, nvalid, wp, m);
  return s_new;
}

template <bool SCALE_BF16>
__device__ __forceinline__ void store_scale(const TensorDesc &td, uint64_t sg, float s) {
  if (SCALE_BF16) static_cast<uint16_t *>(td.s)[sg] = (uint16_t)(f2u(s) >> 16);
  else static_cast<float *>(td.s)[sg] = s;
}

// One lane's 8 consecutive elements, starting at element e0 of tensor td, of which the first nvalid exist;
// scale group number sg; bs_shift = log2(group size) for RED_BLOCK; row = the lane's group within the workgroup for
// RED_WG_ROWS, the first lane of the lane's group for RED_ROWS.  LATE: an earlier kernel of the step has stored v~.
template <int FMT, bool STATE_BF16, bool SCALE_BF16, int ALGO, int ROUND, int ACC, int RED, int CP = CACHED, bool LATE = false>
__device__ __forceinline__ void step_lane(const StepArgs &a, const TensorDesc &td, uint64_t e0, int nvalid,
                                          uint64_t sg, bool scale_writer, uint32_t *slot, int row = 0) {
  constexpr bool ADAM = algo_is_adam(ALGO);
  constexpr bool MASTER = algo_is_master(ALGO);
  constexpr bool KEEP = RED == RED_TILE_KEEP;
  constexpr bool WRITE = RED != RED_TILE && !KEEP;   // the first pass of a two-pass group writes nothing but what is final
  const bool any = ACC == ACC_FULL || nvalid > 0;

  float g[8], m[8], v[8], w[8], x[8], d[8], th[8], sc = 1.0f;
  WavePieces wp = {false, false, 0, e0, nvalid, 0, 0};
  uint32_t c[2] = {0, 0};
  float s_old = 0.0f;
  if (ACC == ACC_FULL || ACC == ACC_LANE) {
    constexpr bool FULL = ACC == ACC_FULL;
    wp = FULL ? full_wave(e0) : wave_pieces(e0, nvalid);
    eco_u32x4_t gq[2] = {}, mq[2] = {}, vq[2] = {}, wq[2] = {};
    if (wp.any_whole) {
      load_wave8<true, FULL, CP>(td.g, wp, gq);
      load_wave8<STATE_BF16, FULL, CP>(td.m, wp, mq);
      if (ADAM) load_wave8<STATE_BF16, FULL, CP>(td.v, wp, vq);
      if (MASTER) {
        load_wave8<false, FULL, CP>(td.aux, wp, wq);
      } else {
        load_codes8<FMT, ACC_FULL, CP>(td.w, wp.from, 8, c);
        uint64_t sl = sg;
        if (!FULL && (RED == RED_BLOCK || RED == RED_ROWS || RED == RED_WG_ROWS)) {
          const uint64_t of_last = (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)sg, wp.last) |
                                   (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(sg >> 32), wp.last) << 32;
          sl = any ? sg : of_last;
        }
        s_old = load_scale<SCALE_BF16>(td.s, sl);
      }
    }
    if (wp.any_cut) {
      if (nvalid & 7) {
        load_ragged8<true>(td.g, e0, nvalid, gq);
        load_ragged8<STATE_BF16>(td.m, e0, nvalid, mq);
        if (ADAM) load_ragged8<STATE_BF16>(td.v, e0, nvalid, vq);
        if (MASTER) {
          load_ragged8<false>(td.aux, e0, nvalid, wq);
        } else {
          load_ragged_codes8<FMT>(td.w, e0, nvalid, c);
          s_old = load_scale<SCALE_BF16>(td.s, sg);
        }
      }
    }
    unpack8<true>(gq, g);
    unpack8<STATE_BF16>(mq, m);
    if (ADAM) unpack8<STATE_BF16>(vq, v);
    if (MASTER) unpack8<false>(wq, w);
  } else {
    load_bf16x8<ACC>(static_cast<const uint16_t *>(td.g) + e0, nvalid, g);
    load_state8<STATE_BF16, ACC>(td.m, e0, nvalid, m);
    if (ADAM) load_state8<STATE_BF16, ACC>(td.v, e0, nvalid, v);
    if (MASTER) {
      load_f32x8<ACC>(static_cast<const float *>(td.aux) + e0, nvalid, w);
    } else {
      load_codes8<FMT, ACC>(td.w, e0, nvalid, c);
      s_old = any ? load_scale<SCALE_BF16>(td.s, sg) : 0.0f;
    }
  }
  if (!MASTER) {
    sc = decode8<FMT>(c, s_old, w);
    if (!exact_scale<SCALE_BF16, ALGO>()) {
#pragma unroll
      for (int j = 0; j < 8; ++j) w[j] *= sc;
    }
  }

  __builtin_amdgcn_s_setprio(0);      // loads issued: back to the default priority (see eco_step_kernel)

  moments_lane<ALGO, LATE>(a, g, m, v, x);
  if (ADAM && (WRITE || KEEP) && !LATE) store_wave8<STATE_BF16, ACC, CP>(td.v, e0, nvalid, wp, v);   // v is final (Alg. 3 returns it unchanged)
  theta_lane<SCALE_BF16, ALGO, ACC>(a, x, w, sc, m, wp.fill, d, th);
  if (KEEP) {
    store_wave8<false, ACC, CP>(td.aux, e0, nvalid, wp, th);
    store_wave8<STATE_BF16, ACC, CP>(td.m, e0, nvalid, wp, m);
  }

  const float amax = group_absmax<RED>(absmax8(th), RED == RED_WG_ROWS || RED == RED_ROWS ? row : (int)td.bs_shift, slot,
                                       RED == RED_ROWS ? (int)(td.group_size >> 3) : RED == RED_WG ? (int)a.wg_waves : 0);
  if (!WRITE) return;
  const Philox4 r = random_lane<ROUND>(a, td, e0, a.seed_lo, a.seed_hi);
  const float s_new = quantize_inject_lane<FMT, STATE_BF16, SCALE_BF16, ALGO, ROUND, ACC, CP>(a, td, e0, nvalid, wp, amax, r, th, d, m);
  if (RED != RED_SLOT && scale_writer && any) store_scale<SCALE_BF16>(td, sg, s_new);
}

// The second pass with master weights: they hold theta~, only the codes are left to write.
template <int FMT, bool SCALE_BF16, int ROUND, int ACC, int CP>
__device__ __forceinline__ void quantize_master_lane(const StepArgs &a, const TensorDesc &td, uint64_t e0, int nvalid, const uint32_t *slot) {
  float th[8], qn[8];
  uint32_t cn[2];
  const WavePieces wp = full_wave(e0);                    // ACC_FULL alone
  if (ACC == ACC_FULL) {
    eco_u32x4_t q[2];
    load_wave8<false, true, CP>(td.aux, wp, q);
    unpack8<false>(q, th);
  } else {
    load_f32x8<ACC>(static_cast<const float *>(td.aux) + e0, nvalid, th);
  }
  const Philox4 r = random_lane<ROUND>(a, td, e0, a.seed_lo, a.seed_hi);
  (void)quantize_lane8<FMT, SCALE_BF16, ROUND, ACC>(u2f(*slot), r, nvalid, th, cn, qn);
  store_wave_codes8<FMT, ACC, CP>(td.w, e0, nvalid, wp, cn);
}

// The launch tables are read-only for the lifetime of a launch; reading them through the constant
// address space lets the compiler fetch them with scalar loads (one per wave, into SGPRs) even
// though the kernel also writes global memory.
#define ECO_CONST_AS __attribute__((address_space(4)))

__device__ __forceinline__ uint32_t load_table(const uint32_t *table, uint32_t i) {
  const ECO_CONST_AS uint32_t *p = (const ECO_CONST_AS uint32_t *)(uintptr_t)table;
  return p[i];
}

__device__ __forceinline__ TensorDesc read_tensor_desc(const ECO_CONST_AS uint64_t *p) {
  TensorDesc td;
  td.w = (void *)(uintptr_t)p[0];
  td.s = (void *)(uintptr_t)p[1];
  td.g = (const void *)(uintptr_t)p[2];
  td.m = (void *)(uintptr_t)p[3];
  td.v = (void *)(uintptr_t)p[4];
  td.aux = (void *)(uintptr_t)p[5];
  td.numel = p[6];
  td.group_size = p[7];
  const uint64_t a8 = p[8], a9 = p[9];
  td.first_unit = (uint32_t)a8;
  td.tensor_id = (uint32_t)(a8 >> 32);
  td.bs_shift = (uint16_t)a9;
  td.kind = (uint16_t)(a9 >> 16);
  td.slot = (uint32_t)(a9 >> 32);
  return td;
}

__device__ __forceinline__ TensorDesc load_tensor_desc(const TensorDesc *tensors, uint32_t ti) {
  return read_tensor_desc((const ECO_CONST_AS uint64_t *)(uintptr_t)(tensors + ti));
}
__device__ __forceinline__ TensorDesc load_tensor_desc(const StepArgs &a, uint32_t ti) { return load_tensor_desc(a.tensors, ti); }

// How many of the 8 elements from e0 on exist before `end`.
__device__ __forceinline__ int valid_from(uint64_t e0, uint64_t end) {
  const int64_t left = (int64_t)end - (int64_t)e0;
  return left >= 8 ? 8 : (left <= 0 ? 0 : (int)left);
}

// ------------------------------------------------------------------ plain optimizer step
// Adam / SGDM on weights that are not quantized.  UNIT_PLAIN_BF16: bf16 weights, result rounded to nearest even, no
// injection (the method is applied to linear layers only; norm weights take the ordinary optimizer).
// UNIT_PLAIN_FP32: fp32 weights under the identity quantizer, for which the quantization error is zero and Alg. 2/3
// add nothing to the momentum.
template <bool W_BF16, bool STATE_BF16, bool ADAM, int ACC, int CP>
__device__ __forceinline__ void plain_lane(const StepArgs &a, const TensorDesc &td, uint64_t e0, int nvalid) {
  constexpr bool FULL = ACC == ACC_FULL;
  float w[8], g[8], m[8], v[8], eta[8];
  const WavePieces wp = FULL ? full_wave(e0) : wave_pieces(e0, nvalid);
  eco_u32x4_t wq[2] = {}, gq[2] = {}, mq[2] = {}, vq[2] = {};
  if (wp.any_whole) {
    load_wave8<W_BF16, FULL, CP>(td.w, wp, wq);
    load_wave8<true, FULL, CP>(td.g, wp, gq);
    load_wave8<STATE_BF16, FULL, CP>(td.m, wp, mq);
    if (ADAM) load_wave8<STATE_BF16, FULL, CP>(td.v, wp, vq);
  }
  if (wp.any_cut) {
    if (nvalid & 7) {
      load_ragged8<W_BF16>(td.w, e0, nvalid, wq);
      load_ragged8<true>(td.g, e0, nvalid, gq);
      load_ragged8<STATE_BF16>(td.m, e0, nvalid, mq);
      if (ADAM) load_ragged8<STATE_BF16>(td.v, e0, nvalid, vq);
    }
  }
  unpack8<W_BF16>(wq, w);
  unpack8<true>(gq, g);
  unpack8<STATE_BF16>(mq, m);
  if (ADAM) unpack8<STATE_BF16>(vq, v);
  if (ADAM) {
    float x[8], d[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      v[j] = fmaf(a.b2, v[j], a.omb2 * (g[j] * g[j]));
      x[j] = v[j] * a.rbc2;
    }
    fill_missing<ACC>(x, wp.fill, 1.0f);
    step_sizes8(a, x, d, eta);
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    float wj = w[j];
    m[j] = fmaf(a.b1, m[j], a.omb1 * g[j]);
    const float u = ADAM ? eta[j] * m[j] : a.lr * m[j];     // the element-wise step size of Sec. 3.2 times the first moment
    if (a.wd != 0.0f) wj = wj - a.wd * wj;
    w[j] = wj - u;
  }
  store_wave8<W_BF16, ACC, CP>(td.w, e0, nvalid, wp, w);
  store_wave8<STATE_BF16, ACC, CP>(td.m, e0, nvalid, wp, m);
  if (ADAM) store_wave8<STATE_BF16, ACC, CP>(td.v, e0, nvalid, wp, v);
}

// ------------------------------------------------------------------ kernels
// One unit of a list of one-wave units (UNIT_*), `lane` in 0..63: what is left beside the full tiles.  One body serves whole
// and partial tiles.
template <int FMT, bool STATE_BF16, bool SCALE_BF16, int ALGO, int ROUND, int CP>
__device__ __forceinline__ void step_wave_unit(const StepArgs &a, const TensorDesc &td, uint32_t unit, uint32_t lane) {
  if (td.kind == UNIT_PLAIN_BF16 || td.kind == UNIT_PLAIN_FP32) {
    const uint64_t e0 = (uint64_t)unit * TILE_ELEMS + (uint64_t)lane * ELEMS_PER_LANE;
    const int nvalid = valid_from(e0, td.numel);
    if (td.kind == UNIT_PLAIN_BF16) plain_lane<true, STATE_BF16, algo_is_adam(ALGO), ACC_LANE, CP>(a, td, e0, nvalid);
    else plain_lane<false, STATE_BF16, algo_is_adam(ALGO), ACC_LANE, CP>(a, td, e0, nvalid);
    return;
  }
  if (td.kind == UNIT_ROWS) {
    // td.slot groups to the wave, one after the other; the lanes beyond them have nothing
    const uint32_t gl = (uint32_t)td.group_size >> 3;                      // lanes of a group: 1..32
    const uint32_t row = (lane * (65536u / gl + 1u)) >> 16;                // lane / gl, exact for lane < 64
    const uint64_t grp = (uint64_t)unit * td.slot;
    const uint64_t e0 = grp * td.group_size + (uint64_t)lane * ELEMS_PER_LANE;
    const uint64_t end = (grp + td.slot) * td.group_size;
    step_lane<FMT, STATE_BF16, SCALE_BF16, ALGO, ROUND, ACC_LANE, RED_ROWS, CP>(
        a, td, e0, valid_from(e0, end < td.numel ? end : td.numel), grp + row, lane == row * gl, nullptr, (int)(row * gl));
    return;
  }
  // a tile, or one group that is reduced like a tile of 512 (bs_shift 9): the segmented reduction above takes six exchanges
  // across lanes, and a wave with one group spends more on them than on its 264 to 504 elements
  const bool row = td.kind == UNIT_ROW;
  const uint64_t start = row ? (uint64_t)unit * td.group_size : (td.kind == UNIT_TAIL ? td.numel / TILE_ELEMS : unit) * TILE_ELEMS;
  const uint64_t end = row && start + td.group_size < td.numel ? start + td.group_size : td.numel;
  const uint64_t e0 = start + (uint64_t)lane * ELEMS_PER_LANE;
  const bool writer = (lane & ((1u << (td.bs_shift - 3)) - 1u)) == 0;
  step_lane<FMT, STATE_BF16, SCALE_BF16, ALGO, ROUND, ACC_LANE, RED_BLOCK, CP>(a, td, e0, valid_from(e0, end), row ? unit : e0 >> td.bs_shift,
                                                                           writer, nullptr);
}

// (1) Block-scaled tensors (group = 32..512 elements, a power of two): one workgroup of one wave per
// full 512-element tile, dispatched in address order.  The tile -> tensor table and the descriptors are
// wave-uniform scalar loads.
// Behind the tiles come the plan's one-wave units: a launch of their own for the norm gains and the ragged tails would
// cost 5-6 us of a step each, whatever they hold.  (No loop over tiles: with one around both bodies the arguments and
// what is derived from them stay live across it and no longer fit the scalar registers.)
// What a wave's way to its data begins with -- the launch's table and the descriptors -- are arguments of their own, in front, here and in
// the kernels below: they are in scalar registers when the wave starts (the build asks for that; members of a struct are not), one
// memory access fewer in a chain of four (one matrix of 1 M elements 5.2 -> 5.0 us, of 4 M 16.9 -> 16.7).  As integers: for every argument
// of pointer type the runtime looks up the allocation behind it, 0.03 us of a call each.  `table` also covers the one-wave units, whose list
// lies behind the tiles'.  FP8, bf16 state, fp32 scales, Adam and nearest rounding take 65 registers, here and in the wide kernel with one-wave units,
// so seven waves a SIMD; held to 64 they run eight, which is no faster (us, 65 / 64: 4 M elements 8.70 / 8.79, 8 M 18.69 / 19.01, 16 M 30.7 / 31.0,
// 21 M 40.3 / 40.7; rows of 200 12.04 / 12.05; 5.7 M 13.16 / 12.94).
template <int FMT, bool STATE_BF16, bool SCALE_BF16, int ALGO, int ROUND, int CP>
__global__ __launch_bounds__(WG_THREADS) void eco_step_kernel(const uint64_t table, const uint64_t tensors, const StepArgs a) {
  // A wave that has not issued its loads yet goes first: its address arithmetic and load instructions
  // are not queued behind the arithmetic of the waves that already have their data (the priority is
  // dropped again in step_lane, once the loads are issued).  Measured: +0.3 % and a flatter optimum
  // over the occupancy cap.
  __builtin_amdgcn_s_setprio(3);
  const TensorDesc td = load_tensor_desc((const TensorDesc *)tensors, load_table((const uint32_t *)table, blockIdx.x));
  const uint32_t tile = blockIdx.x + a.unit_base;
  if (tile < a.num_tiles) {
    const uint64_t e0 = (uint64_t)(tile - td.first_unit) * TILE_ELEMS + (uint64_t)threadIdx.x * ELEMS_PER_LANE;
    const bool writer = (threadIdx.x & ((1u << (td.bs_shift - 3)) - 1u)) == 0;
    step_lane<FMT, STATE_BF16, SCALE_BF16, ALGO, ROUND, ACC_FULL, RED_BLOCK, CP>(a, td, e0, 8, e0 >> td.bs_shift, writer, nullptr);
  } else {
    step_wave_unit<FMT, STATE_BF16, SCALE_BF16, ALGO, ROUND, CP>(a, td, tile - a.num_tiles - td.first_unit, threadIdx.x);
  }
}

// (2) Wide groups (any multiple of 8 from 520 to 8192 elements: row-wise scaling, Sec. 4.1): one workgroup of
// ceil(group/512) waves per group, abs-max by wave all-reduce plus an LDS combine across the waves -- or one workgroup
// per bundle of 2..8 groups (TensorDesc::slot), which fill a whole number of waves exactly (wide_geometry) or leave
// lanes of the last one idle (step_geometry).  EXTRA: workgroups beyond the groups take one-wave units, one
// to a wave (a variant of its own: with those paths in the kernel the groups run 3.6 % slower, 3 460 -> 3 590 us over
// Gemma-3-1B shapes, so a long launch leaves them to another one).
template <int FMT, bool STATE_BF16, bool SCALE_BF16, int ALGO, int ROUND, bool EXTRA, int CP>
__global__ __launch_bounds__(1024) void eco_step_wide_kernel(const uint64_t table, const uint64_t tensors, const StepArgs a) {
  __builtin_amdgcn_s_setprio(3);      // as in eco_step_kernel: loading waves first
  const uint32_t unit = blockIdx.x + a.unit_base;
  if (EXTRA && unit >= a.num_units) {
    const uint32_t x = __builtin_amdgcn_readfirstlane((unit - a.num_units) * a.wg_waves + (threadIdx.x >> 6));
    if (x < a.num_extra) {
      const TensorDesc td = load_tensor_desc(a, load_table(a.extra_tensor, x));
      step_wave_unit<FMT, STATE_BF16, SCALE_BF16, ALGO, ROUND, CP>(a, td, x - td.first_unit, threadIdx.x & 63);
    }
    return;
  }
  const TensorDesc td = load_tensor_desc((const TensorDesc *)tensors, load_table((const uint32_t *)table, blockIdx.x));
  const uint32_t rows = td.slot;
  const uint64_t grp = (uint64_t)(unit - td.first_unit) * rows;       // the workgroup's first group
  const uint64_t start = grp * td.group_size;
  const uint32_t lane_elem = threadIdx.x * ELEMS_PER_LANE;
  const uint64_t e0 = start + lane_elem;
  const uint64_t end = start + rows * td.group_size < td.numel ? start + rows * td.group_size : td.numel;
  if (rows > 1) {
    const uint32_t gs = (uint32_t)td.group_size;
    uint32_t row = 0;
    for (uint32_t k = 1; k < rows; ++k) row += lane_elem >= k * gs ? 1u : 0u;
    if (ALGO == ALGO_ADAM_MASTER || end - start == (uint64_t)a.wg_waves * TILE_ELEMS)      // master weights: see step_geometry
      step_lane<FMT, STATE_BF16, SCALE_BF16, ALGO, ROUND, ACC_FULL, RED_WG_ROWS, CP>(a, td, e0, 8, grp + row, lane_elem == row * gs, nullptr,
                                                                                 (int)row);
    else
      step_lane<FMT, STATE_BF16, SCALE_BF16, ALGO, ROUND, ACC_LANE, RED_WG_ROWS, CP>(a, td, e0, valid_from(e0, end), grp + row,
                                                                                 lane_elem == row * gs, nullptr, (int)row);
    return;
  }
  // a group that fills every lane of the workgroup (e.g. rows of 1024, 2048, 4096) needs no per-lane guards
  if (end - start == (uint64_t)a.wg_waves * TILE_ELEMS)
    step_lane<FMT, STATE_BF16, SCALE_BF16, ALGO, ROUND, ACC_FULL, RED_WG, CP>(a, td, e0, 8, grp, threadIdx.x == 0, nullptr);
  else
    step_lane<FMT, STATE_BF16, SCALE_BF16, ALGO, ROUND, ACC_LANE, RED_WG, CP>(a, td, e0, valid_from(e0, end), grp,
                                                                          threadIdx.x == 0, nullptr);
}

// (3) Lists of little work, every class of scale group but the long tensor-wise one in one launch: a step of small tensors is
// bound by launches (2.6 us of host time each, 4-6 us on the device with the drain between two), not by what they do.  All
// workgroups have the waves that the widest group asks for (wg_waves).  Groups wider than a wave are packed as many units to a
// workgroup as its waves hold; one-wave units take a wave each.  wg: the workgroup's number within its tensor.
template <int FMT, bool STATE_BF16, bool SCALE_BF16, int ALGO, int ROUND>
__device__ __forceinline__ void step_list_workgroup(const StepArgs &a, const TensorDesc &td, uint32_t wg) {
  const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nwaves = a.wg_waves;
  const uint32_t gs = (uint32_t)td.group_size, rows = td.slot;
  if (td.kind != UNIT_WIDE) {
    const uint32_t unit = wg * nwaves + wave;
    if ((uint64_t)unit * (td.kind == UNIT_ROWS ? rows * gs : td.kind == UNIT_ROW ? gs : (uint32_t)TILE_ELEMS) >= td.numel) return;
    const uint64_t tile_off = (uint64_t)unit * TILE_ELEMS;
    if (td.kind == UNIT_TILES && tile_off + TILE_ELEMS <= td.numel) {
      const uint64_t e0 = tile_off + (uint64_t)lane * ELEMS_PER_LANE;
      const bool writer = (lane & ((1u << (td.bs_shift - 3)) - 1u)) == 0;
      step_lane<FMT, STATE_BF16, SCALE_BF16, ALGO, ROUND, ACC_FULL, RED_BLOCK>(a, td, e0, 8, e0 >> td.bs_shift, writer, nullptr);
    } else {
      step_wave_unit<FMT, STATE_BF16, SCALE_BF16, ALGO, ROUND, CACHED>(a, td, unit, lane);
    }
    return;
  }
  const uint32_t uw = (rows * gs + TILE_ELEMS - 1) / TILE_ELEMS, per_wg = nwaves / uw;   // waves of a unit, units of a workgroup
  const uint32_t u = wave / uw, unit = wg * per_wg + u;
  const uint32_t lane_elem = (wave - u * uw) * TILE_ELEMS + lane * ELEMS_PER_LANE;
  const uint64_t start = (uint64_t)unit * rows * gs;
  uint64_t end = start + (uint64_t)rows * gs < td.numel ? start + (uint64_t)rows * gs : td.numel;
  if (u >= per_wg || start >= td.numel) end = 0;          // nothing to do, but the barriers are the workgroup's
  uint32_t row = 0;
  for (uint32_t k = 1; k < rows; ++k) row += lane_elem >= k * gs ? 1u : 0u;
  step_lane<FMT, STATE_BF16, SCALE_BF16, ALGO, ROUND, ACC_LANE, RED_WG_ROWS>(
      a, td, start + lane_elem, valid_from(start + lane_elem, end), (uint64_t)unit * rows + row, lane_elem == row * gs, nullptr,
      u < per_wg ? (int)(u * rows + row) : 0);
}

// 64 registers at most, for eight waves a SIMD: with 65, as FP8 with Adam had, seven (us, 65 / 64: rows of 576, 5.5 M elements with fp32
// state 26.6 / 24.3, with bf16 state 22.6 / 19.7).
// With the descriptors in the kernel arguments (no table in device memory); a workgroup finds its tensor by comparing its number
// with the tensors' first ones, a lane each.
template <int FMT, bool STATE_BF16, bool SCALE_BF16, int ALGO, int ROUND>
__global__ __launch_bounds__(1024, 8) void eco_step_small_kernel(const SmallArgs args) {
  const ECO_CONST_AS SmallArgs *ka = (const ECO_CONST_AS SmallArgs *)__builtin_amdgcn_kernarg_segment_ptr();
  __builtin_amdgcn_s_setprio(3);
  const uint32_t lane = threadIdx.x & 63;
  const uint32_t first = lane < args.num ? ka->first_wg[lane] : 0xFFFFFFFFu;
  const uint32_t ti = (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(first <= blockIdx.x)) - 1u;
  const TensorDesc td = read_tensor_desc((const ECO_CONST_AS uint64_t *)&ka->desc[ti]);
  step_list_workgroup<FMT, STATE_BF16, SCALE_BF16, ALGO, ROUND>(args.step, td, blockIdx.x - ka->first_wg[ti]);
}

// With a plan's tables: any number of tensors (415 of them in rows of 984, 3024, 1120 and 4856 elements, us: a launch for each number of
// waves 19.7, this 7.9; 142 in rows of 2304 and 108 in rows of 512 20.3 / 12.3).
template <int FMT, bool STATE_BF16, bool SCALE_BF16, int ALGO, int ROUND>
__global__ __launch_bounds__(1024, 8) void eco_step_list_kernel(const uint64_t table, const uint64_t tensors, const StepArgs a) {
  __builtin_amdgcn_s_setprio(3);
  const TensorDesc td = load_tensor_desc((const TensorDesc *)tensors, load_table((const uint32_t *)table, blockIdx.x));
  step_list_workgroup<FMT, STATE_BF16, SCALE_BF16, ALGO, ROUND>(a, td, blockIdx.x + a.unit_base - td.first_unit);
}

// (4) One scale per tensor (tensor-wise scaling, Sec. 4.4), tensors too large for one workgroup: two passes
// over 512-element tiles.  Pass 1 recomputes theta~ and leaves each tile's abs-max in a scratch array, which
// a reduction kernel (see eco_tensorwise_reduce_kernel) folds into the tensor's slot; pass 2 recomputes theta~ again
// (the inputs are untouched so far), quantizes against the slot's value and writes codes and state; a last
// kernel writes the new scales.  With master weights nothing but the codes waits for the scale: pass 1 stores them and the
// moments, pass 2 reads them alone (31 bytes a parameter with Adam and fp32 state where recomputing takes 41: six tensors of 64 M
// elements in INT4 2817 -> 2164 us; SGDM 324 M 1644 -> 1295; Adam with bf16 state two of 51 M 544 -> 415).
template <int FMT, bool STATE_BF16, bool SCALE_BF16, int ALGO, int ROUND, int RED, int CP>
__global__ __launch_bounds__(WG_THREADS) void eco_step_tensorwise_kernel(const StepArgs a) {
  __builtin_amdgcn_s_setprio(3);      // as in eco_step_kernel: loading waves first
  // Pass 2 goes through the tiles backwards, each on the XCD that has it in its L2 from pass 1 (us, forwards / backwards by single tiles,
  // which takes every tile to another XCD / this: FP8 with fp32 state 1 M elements 14.7 / 17.6 / 14.4, 4 M 32.6 / 31.4 / 27.7, 8 M 51.7 /
  // 49.8 / 45.4, two of 60 M 660 / 639 / 634; INT4 with bf16 state 2.2 M in seven tensors 16.0 / 20.0 / 16.1, 7 M 34.2 / 34.1 / 30.1, 210 M
  // 622 / 600 / 599).
  const uint32_t nth = blockIdx.x + a.unit_base, unit = RED == RED_SLOT ? backwards_on_the_same_xcd(nth, a.num_tw_tiles) : nth;
  const TensorDesc td = load_tensor_desc(a, load_table(a.tw_tile_tensor, unit));
  const uint64_t tile_off = (uint64_t)(unit - td.first_unit) * TILE_ELEMS;
  const uint64_t e0 = tile_off + (uint64_t)threadIdx.x * ELEMS_PER_LANE;
  uint32_t *slot = RED == RED_TILE ? a.tile_max + unit : a.slots + td.slot;
  constexpr int R = algo_is_master(ALGO) && RED == RED_TILE ? RED_TILE_KEEP : RED;
  const bool whole = tile_off + TILE_ELEMS <= td.numel;
  const int nvalid = valid_from(e0, td.numel);
  if (algo_is_master(ALGO) && RED == RED_SLOT) {
    if (whole) quantize_master_lane<FMT, SCALE_BF16, ROUND, ACC_FULL, CP>(a, td, e0, 8, slot);
    else quantize_master_lane<FMT, SCALE_BF16, ROUND, ACC_GUARDED, CACHED>(a, td, e0, nvalid, slot);
  } else if (whole) {
    step_lane<FMT, STATE_BF16, SCALE_BF16, ALGO, ROUND, ACC_FULL, R, CP>(a, td, e0, 8, 0, false, slot);
  } else {
    step_lane<FMT, STATE_BF16, SCALE_BF16, ALGO, ROUND, ACC_GUARDED, R>(a, td, e0, nvalid, 0, false, slot);
  }
}

// tw_reduce_wgs workgroups per tensor (one for every 16 384 tiles of the longest), which meet in its slot (zero until
// then; the scale kernel leaves it so): one alone took 158 us over the 409 600 tiles of an embedding, a serial read of
// 1.6 MB; 26 take 6 us.
constexpr int TW_REDUCE_THREADS = 1024;
template <int FMT>   // a template only so that every translation unit may hold its own copy
__global__ __launch_bounds__(TW_REDUCE_THREADS) void eco_tensorwise_reduce_kernel(const StepArgs a) {
  const uint32_t unit = blockIdx.x + a.unit_base;
  const TensorDesc td = load_tensor_desc(a, a.tw_tensor[unit / a.tw_reduce_wgs]);
  const uint64_t ntiles = (td.numel + TILE_ELEMS - 1) / TILE_ELEMS;
  const uint64_t first = (uint64_t)(unit % a.tw_reduce_wgs) * TW_REDUCE_THREADS;
  if (first >= ntiles) return;
  const uint32_t *tm = a.tile_max + td.first_unit;
  uint32_t r = 0;
  for (uint64_t i = first + threadIdx.x; i < ntiles; i += (uint64_t)TW_REDUCE_THREADS * a.tw_reduce_wgs) { const uint32_t x = tm[i]; r = r > x ? r : x; }
  r = group_umax(r, 64);
  __shared__ uint32_t wave_max[TW_REDUCE_THREADS / 64];
  if ((threadIdx.x & 63) == 0) wave_max[threadIdx.x >> 6] = r;
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int k = 1; k < TW_REDUCE_THREADS / 64; ++k) { const uint32_t o = wave_max[k]; r = r > o ? r : o; }
    atomicMax(&a.slots[td.slot], r);
  }
}

template <int FMT, bool SCALE_BF16>
__global__ __launch_bounds__(WG_THREADS) void eco_tensorwise_scale_kernel(const StepArgs a) {
  const uint32_t i = (blockIdx.x + a.unit_base) * WG_THREADS + threadIdx.x;
  if (i >= a.num_tw_tensors) return;
  const TensorDesc td = load_tensor_desc(a, a.tw_tensor[i]);
  float s_new, inv;
  block_scale<FMT, SCALE_BF16>(u2f(a.slots[td.slot]), s_new, inv);
  store_scale<SCALE_BF16>(td, 0, s_new);
  a.slots[td.slot] = 0;
}

// Every launch is followed by its own error check, so that a failed launch stops the sequence and is the
// error that is reported.
#define ECO_LAUNCH_CHECKED(kernel, grid, block, lds, stream, ...)                                                 \
  do {                                                                                                            \
    hipLaunchKernelGGL(kernel, grid, block, lds, stream, __VA_ARGS__);                                            \
    const hipError_t launch_err_ = hipGetLastError();                                                             \
    if (launch_err_ != hipSuccess) return launch_err_;                                                            \
  } while (0)

// One work item per workgroup, `units` of them: as many launches as the limit on the threads of one launch asks
// for (the runtime wants grid x block below 2^32), each told where it starts through StepArgs::unit_base.
template <class Kernel>
hipError_t launch_in_chunks(Kernel kernel, uint64_t units, unsigned block, unsigned lds, hipStream_t stream, StepArgs args,
                            uint64_t max_launch_threads) {
  const uint64_t per_launch = max_launch_threads / block ? max_launch_threads / block : 1;
  for (uint64_t base = 0; base < units; base += per_launch) {
    args.unit_base = static_cast<uint32_t>(base);
    const uint64_t n = units - base < per_launch ? units - base : per_launch;
    ECO_LAUNCH_CHECKED(kernel, dim3(static_cast<unsigned>(n)), dim3(block), lds, stream, args);
  }
  return hipSuccess;
}
// The same for a kernel that takes its table, from the launch's first work item on, and the descriptors as arguments of their own.
template <class Kernel>
hipError_t launch_listed_in_chunks(Kernel kernel, const uint32_t *table, uint64_t units, unsigned block, unsigned lds, hipStream_t stream,
                                   StepArgs args, uint64_t max_launch_threads) {
  const uint64_t per_launch = max_launch_threads / block ? max_launch_threads / block : 1;
  for (uint64_t base = 0; base < units; base += per_launch) {
    const uint64_t n = units - base < per_launch ? units - base : per_launch;
    args.unit_base = static_cast<uint32_t>(base);
    ECO_LAUNCH_CHECKED(kernel, dim3(static_cast<unsigned>(n)), dim3(block), lds, stream, reinterpret_cast<uint64_t>(table + base),
                       reinterpret_cast<uint64_t>(args.tensors), args);
  }
  return hipSuccess;
}
#define ECO_LISTED_CHECKED(...)                                         \
  do {                                                                  \
    const hipError_t chunk_err_ = launch_listed_in_chunks(__VA_ARGS__); \
    if (chunk_err_ != hipSuccess) return chunk_err_;                    \
  } while (0)
#define ECO_CHUNKS_CHECKED(...)                                  \
  do {                                                           \
    const hipError_t chunk_err_ = launch_in_chunks(__VA_ARGS__); \
    if (chunk_err_ != hipSuccess) return chunk_err_;             \
  } while (0)

template <int FMT, bool STATE_BF16, bool SC, int RD, int AL>
hipError_t launch_resident(const StepLaunch &sl, hipStream_t stream);      // eco_step_resident.hpp

// Full tiles and one-wave units.
template <int FMT, bool STATE_BF16, bool SC, int RD, int AL, int CP>
hipError_t launch_tiles(const StepLaunch &sl, hipStream_t stream) {
  StepArgs ta = sl.args;
  if (sl.extra_in != 0) ta.num_extra = 0;
  ECO_LISTED_CHECKED((eco_step_kernel<FMT, STATE_BF16, SC, AL, RD, CP>), sl.tile_tensor, (uint64_t)ta.num_tiles + ta.num_extra, WG_THREADS,
                     sl.lds_bytes, stream, ta, sl.max_tile_threads);
  return hipSuccess;
}
// The wide groups whose workgroups have nw waves.
template <int FMT, bool STATE_BF16, bool SC, int RD, int AL, int CP>
hipError_t launch_wide(const StepLaunch &sl, int nw, hipStream_t stream) {
  StepArgs wa = sl.args;
  const unsigned lds = sl.lds_bytes_wide[nw];
  const uint32_t *const table = sl.wide_base + sl.wide_offset[nw];
  const uint32_t units = wa.num_units = sl.num_wide[nw];
  wa.wg_waves = static_cast<uint32_t>(nw);
  if (sl.extra_in != nw || !wa.num_extra)
    ECO_LISTED_CHECKED((eco_step_wide_kernel<FMT, STATE_BF16, SC, AL, RD, false, CP>), table, units, 64 * nw, lds, stream, wa,
                       sl.max_launch_threads);
  else
    ECO_LISTED_CHECKED((eco_step_wide_kernel<FMT, STATE_BF16, SC, AL, RD, true, CP>), table, (uint64_t)units + (wa.num_extra + nw - 1) / nw,
                       64 * nw, lds, stream, wa, sl.max_launch_threads);
  return hipSuccess;
}

// The two passes of tensor-wise scaling with the reduction between them.  Past the caches (us): 210 M elements, INT4 601 -> 572, FP8 1109 -> 1020,
// with master weights 1204 -> 1099; 20 M (220 MB in FP8) would lose, 95 -> 104.
template <int FMT, bool STATE_BF16, bool SC, int RD, int AL, int CP>
hipError_t launch_two_passes(const StepLaunch &sl, hipStream_t stream) {
  const StepArgs &args = sl.args;
  ECO_CHUNKS_CHECKED((eco_step_tensorwise_kernel<FMT, STATE_BF16, SC, AL, RD, RED_TILE, CP>), args.num_tw_tiles, WG_THREADS,
                     sl.lds_bytes_tw, stream, args, sl.max_launch_threads);
  ECO_CHUNKS_CHECKED((eco_tensorwise_reduce_kernel<FMT>), (uint64_t)args.num_tw_tensors * args.tw_reduce_wgs, TW_REDUCE_THREADS, 0, stream,
                     args, sl.max_launch_threads);
  ECO_CHUNKS_CHECKED((eco_step_tensorwise_kernel<FMT, STATE_BF16, SC, AL, RD, RED_SLOT, CP>), args.num_tw_tiles, WG_THREADS,
                     sl.lds_bytes_tw, stream, args, sl.max_launch_threads);
  return hipSuccess;
}

template <int FMT, bool STATE_BF16, bool SC, int RD, int AL>
hipError_t launch_step_kernels(const StepLaunch &sl, hipStream_t stream) {
  const StepArgs &args = sl.args;
  if (sl.small) {
    ECO_LAUNCH_CHECKED((eco_step_small_kernel<FMT, STATE_BF16, SC, AL, RD>), dim3((unsigned)sl.list_wgs), dim3(64 * sl.list_waves), 0, stream,
                       *sl.small);
  } else if (sl.list_wgs) {
    StepArgs la = args;
    la.wg_waves = sl.list_waves;
    ECO_LISTED_CHECKED((eco_step_list_kernel<FMT, STATE_BF16, SC, AL, RD>), sl.list_tensor, sl.list_wgs, 64 * sl.list_waves, 0, stream, la,
                       sl.max_launch_threads);
  } else {
    if (args.num_tiles || (args.num_extra && sl.extra_in == 0)) {
      const hipError_t e = sl.stream & 1u ? launch_tiles<FMT, STATE_BF16, SC, RD, AL, STREAM_WAVE>(sl, stream)
                                          : launch_tiles<FMT, STATE_BF16, SC, RD, AL, CACHED>(sl, stream);
      if (e != hipSuccess) return e;
    }
    for (int nw = 1; nw <= MAX_WIDE_WAVES; ++nw) {
      if (!sl.num_wide[nw]) continue;
      const hipError_t e = sl.stream >> nw & 1u ? launch_wide<FMT, STATE_BF16, SC, RD, AL, STREAM_GROUP>(sl, nw, stream)
                                                : launch_wide<FMT, STATE_BF16, SC, RD, AL, CACHED>(sl, nw, stream);
      if (e != hipSuccess) return e;
    }
  }
  if (args.num_slabs) {
    const hipError_t e = launch_resident<FMT, STATE_BF16, SC, RD, AL>(sl, stream);
    if (e != hipSuccess) return e;
  }
  if (args.num_tw_tiles) {
    const hipError_t e = sl.stream >> STREAM_TENSORWISE & 1u ? launch_two_passes<FMT, STATE_BF16, SC, RD, AL, STREAM_GROUP>(sl, stream)
                                                             : launch_two_passes<FMT, STATE_BF16, SC, RD, AL, CACHED>(sl, stream);
    if (e != hipSuccess) return e;
    ECO_CHUNKS_CHECKED((eco_tensorwise_scale_kernel<FMT, SC>), (args.num_tw_tensors + WG_THREADS - 1) / WG_THREADS, WG_THREADS,
                       0, stream, args, sl.max_launch_threads);
  }
  return hipSuccess;
}

template <int FMT, bool STATE_BF16, bool SC, int RD>
hipError_t launch_step_algos(const KernelVariant &kv, const StepLaunch &sl, hipStream_t stream) {
  switch (kv.algo) {
    case ALGO_ADAM: return launch_step_kernels<FMT, STATE_BF16, SC, RD, ALGO_ADAM>(sl, stream);
    case ALGO_SGDM: return launch_step_kernels<FMT, STATE_BF16, SC, RD, ALGO_SGDM>(sl, stream);
    case ALGO_SGDM_EXACT: return launch_step_kernels<FMT, STATE_BF16, SC, RD, ALGO_SGDM_EXACT>(sl, stream);
    case ALGO_ADAM_MASTER: return launch_step_kernels<FMT, STATE_BF16, SC, RD, ALGO_ADAM_MASTER>(sl, stream);
    default: return launch_step_kernels<FMT, STATE_BF16, SC, RD, ALGO_SGDM_MASTER>(sl, stream);
  }
}

template <int FMT, bool STATE_BF16>
hipError_t launch_step_variants(const KernelVariant &kv, const StepLaunch &sl, hipStream_t stream) {
  const int key = (kv.scale_bf16 ? 2 : 0) | (kv.round == ROUND_RTN ? 1 : 0);
  switch (key) {
    case 0: return launch_step_algos<FMT, STATE_BF16, false, ROUND_SR>(kv, sl, stream);
    case 1: return launch_step_algos<FMT, STATE_BF16, false, ROUND_RTN>(kv, sl, stream);
    case 2: return launch_step_algos<FMT, STATE_BF16, true, ROUND_SR>(kv, sl, stream);
    default: return launch_step_algos<FMT, STATE_BF16, true, ROUND_RTN>(kv, sl, stream);
  }
}

}  // namespace eco
