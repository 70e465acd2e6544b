// Tensor-wise scaling (Sec. 4.4) in one pass over memory: tensors that the chip can hold.
//
// One scale for a tensor means that no element can be quantized before every element's theta~ is known.  The two-pass
// form (eco_step_tensorwise_kernel) recomputes theta~ and reads the inputs twice, 31 bytes a parameter instead of 20 in
// FP8 with fp32 state, 17.5 instead of 11 in INT4 with bf16 state.  The register files and LDS of 256 compute units hold
// 12 bytes (theta~, m~, d) for 8 million elements, so here they wait on the chip for the tensor's maximum instead:
//
// The tensors of the list, one after the other, are cut into slabs of 6144 elements (one 512-element tile to each of a
// workgroup's 12 waves).  One workgroup per compute unit takes every resident_wgs-th slab.  In turn i a wave computes theta~ of
// its tile of slab i, keeps it, and the workgroup publishes the slab's maximum in slab_max[]; then it quantizes and
// writes its tile of slab i - 4, whose tensor's last slab has been published by some workgroup a turn or more ago.  The
// loads of slab i + 1 are in flight all the while, and the entries of slab_max[] that the next turn needs are loaded a
// turn ahead, so neither memory nor the exchange between compute units is waited for in the steady state.
//
// Nothing depends on the workgroups being resident together: a wait for entries is a bounded number of reads.  A
// workgroup that gives up marks its slab and goes on (at most fp32 v~ has been stored, everything else the slab needs is
// still in place), and a second kernel finishes marked slabs from memory.  That kernel also writes the new scales (until
// then the old ones are there for marked slabs) and empties slab_max[] for the next step.  (Giving up is no rarity: a
// workgroup takes a whole compute unit, so with a kernel of another stream on the chip some come late.  A store to the
// slab's own flag is all that it costs: a list with an atomic counter was 10 000 additions to one address for each 5 M
// elements.)
//
// Progress and reuse inside a workgroup, without barriers: a wave contributes to an "event" (the resolution of a
// tensor's maximum: each lane reads one of the entries) and waits for the other waves.  They never wait for it in turn:
// the wave that is furthest behind waits only for contributions that the others have made.  Between two events lie
// fewer turns than slabs are in hand (a resolved tensor has no slab beyond those), and without a maximum there is an
// event every turn, so waves are never RES_RING turns apart and an entry of the rings is not reused before all have
// left it.
//
// What bounds it: memory for fp32 state (5.2 of the 6.1 TB/s of the block-scaled form); for INT4 with bf16 state the
// vector ALU's issue beside it (see the counters in profiles/).  Measured, two-pass form -> this one, 369 M elements in
// tensors of 1408 x 2048: FP8, fp32 state 1964 -> 1430 us; INT4, bf16 state 1112 -> 872 us; three tensors of 40 000
// elements 14.2 -> 12.8 us; past the caches (CP, see there) 1153 M in tensors of that kind FP8 4378 -> 3820 and INT4 2492 -> 2412; where a list is too short for it or has company that costs launches, see one_pass_pays.  What
// it took: 12 waves of 168 registers rather than 8 of 256 (INT4 1290 -> 1000 us), no memory access inside a branch (1000 ->
// 940), an event's contributions half a turn before the result is wanted (940 -> 890).  19 of the 80 variants, among them
// Adam with bf16 state and stochastic rounding, do not quite fit 168 registers and keep 2 to 11 values in scratch memory, and so do 15 of the 80 that pass the
// caches by; all of these are as fast as the two forms before them or faster (721 M elements in tensors of 1408 x 2048, one each, through the
// caches before waves took whole lines / past them: FP8, Adam with master weights 3774 / 3287, INT4, bf16 state, Adam 1569 / 1529, SGDM 1123 / 1125).
#pragma once
#include "eco_step_kernel.hpp"

namespace eco {

constexpr int RES_RING = 16;           // LDS entries for slabs whose maximum is being collected
static_assert(RES_RING >= 2 * RES_DEPTH, "resident step rings");
constexpr uint32_t NO_MAX = 0xFFFFFFFFu;       // an entry of slab_max[] that has not been published (no maximum has the sign bit)

// Memory access of a wave's tile: buffer instructions, whose hardware bound drops what lies beyond the tensor's end -- or
// everything, where there is no tile to load or store.  No access then stands inside a branch.  That matters: loads and
// stores count in one counter, in order, and a wait for loads whose number of younger stores depends on the path taken
// has to drain the stores as well, about 1.5 us a turn.  (Nor are they FLAT instructions, which count as LDS operations
// too, so that every wait for an LDS result or a scalar load would wait for the tile in flight.)
__device__ __forceinline__ buffer_t tile_buffer(const void *array, uint64_t tile, uint32_t len, uint32_t elem_bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(static_cast<const char *>(array)) + tile * elem_bytes, 0,
                                           (int)(len * elem_bytes), 0x00020000);
}
template <int CP>
__device__ __forceinline__ eco_u32x4_t load16(buffer_t b, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b128(b, off, 0, CP != CACHED ? POLICY_NT : 0);
}
template <int CP>
__device__ __forceinline__ void store16(buffer_t b, uint32_t off, eco_u32x4_t x) { __builtin_amdgcn_raw_buffer_store_b128(x, b, off, 0, CP); }
__device__ __forceinline__ eco_u32x4_t bits4(const float *x) { return eco_u32x4_t{f2u(x[0]), f2u(x[1]), f2u(x[2]), f2u(x[3])}; }
constexpr int SCOPE_AGENT = 16;        // cache policy: coherent between the XCDs

// Eight fp32 of each lane: past the caches in whole lines to an instruction (see exchange_chunks, which a load still needs once it has
// arrived); from the cache 32 bytes to a lane, without the exchange on a short step's way (1 M elements 13.4 us, with it 14.0).
template <int CP>
__device__ __forceinline__ void load_f32_tile(buffer_t b, eco_u32x4_t (&q)[2]) {
  q[0] = load16<CP>(b, CP != CACHED ? lane_chunk() * 16 : (threadIdx.x & 63) * 32);
  q[1] = load16<CP>(b, CP != CACHED ? lane_chunk() * 16 + 1024 : (threadIdx.x & 63) * 32 + 16);
}
template <int CP>
__device__ __forceinline__ void store_f32_tile(buffer_t b, const float (&x)[8]) {
  eco_u32x4_t q[2] = {bits4(x), bits4(x + 4)};
  if (CP != CACHED) exchange_chunks(q);
  store16<CP>(b, CP != CACHED ? lane_chunk() * 16 : (threadIdx.x & 63) * 32, q[0]);
  store16<CP>(b, CP != CACHED ? lane_chunk() * 16 + 1024 : (threadIdx.x & 63) * 32 + 16, q[1]);
}
template <bool BF16, int CP>
__device__ __forceinline__ void unpack_tile(eco_u32x4_t (&q)[2], float (&x)[8]) {
  if (!BF16 && CP != CACHED) exchange_chunks(q);
  unpack8<BF16>(q, x);
}
template <bool BF16, int CP>
__device__ __forceinline__ void store_state_tile(void *array, uint64_t tile, uint32_t len, uint32_t lane, const float (&x)[8]) {
  const buffer_t b = tile_buffer(array, tile, len, BF16 ? 2 : 4);
  if (BF16) store16<CP>(b, lane * 16, pack_bf16x8(x));
  else store_f32_tile<CP>(b, x);
}

// What a lane loads for a tile, as it comes from memory.
template <int FMT, bool STATE_BF16, int ALGO>
struct RawLane {
  uint32_t c[2];
  float s;
  eco_u32x4_t g, m[2], v[2], w[2];
};

template <int FMT, bool STATE_BF16, bool SCALE_BF16, int ALGO, int CP>
__device__ __forceinline__ void load_raw(const TensorDesc &td, uint64_t tile, uint32_t len, uint32_t lane, RawLane<FMT, STATE_BF16, ALGO> &r) {
  constexpr uint32_t ES = STATE_BF16 ? 2 : 4;
  r.g = load16<CP>(tile_buffer(td.g, tile, len, 2), lane * 16);
  const buffer_t bm = tile_buffer(td.m, tile, len, ES);
  if (STATE_BF16) r.m[0] = load16<CP>(bm, lane * 16);
  else load_f32_tile<CP>(bm, r.m);
  if (algo_is_adam(ALGO)) {
    const buffer_t bv = tile_buffer(td.v, tile, len, ES);
    if (STATE_BF16) r.v[0] = load16<CP>(bv, lane * 16);
    else load_f32_tile<CP>(bv, r.v);
  }
  if (algo_is_master(ALGO)) {
    load_f32_tile<CP>(tile_buffer(td.aux, tile, len, 4), r.w);
    r.s = 0.0f;
  } else {
    if (FMT == FMT_FP8) {
      const eco_u32x2_t c = __builtin_amdgcn_raw_buffer_load_b64(tile_buffer(td.w, tile, len, 1), lane * 8, 0, CP != CACHED ? POLICY_NT : 0);
      r.c[0] = c.x; r.c[1] = c.y;
    } else {
      r.c[0] = __builtin_amdgcn_raw_buffer_load_b32(tile_buffer(td.w, tile >> 1, len >> 1, 1), lane * 4, 0, CP != CACHED ? POLICY_NT : 0);
      r.c[1] = 0;
    }
    r.s = SCALE_BF16 ? u2f((uint32_t)__builtin_amdgcn_raw_buffer_load_b16(tile_buffer(td.s, 0, 1, 2), 0, 0, 0) << 16)
                     : u2f(__builtin_amdgcn_raw_buffer_load_b32(tile_buffer(td.s, 0, 1, 4), 0, 0, 0));
  }
}

// LDS words shared by the waves of a workgroup.  The hardware executes a compute unit's LDS operations of one wave in
// order; the empty asm statements keep the compiler to it.
__device__ __forceinline__ uint32_t lds_read(const uint32_t *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_write(uint32_t *p, uint32_t x) {
  __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ void lds_max(uint32_t *p, uint32_t x) {
  (void)__hip_atomic_fetch_max(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}
__device__ __forceinline__ uint32_t lds_add1(uint32_t *p) {
  asm volatile("" ::: "memory");
  const uint32_t old = __hip_atomic_fetch_add(p, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  asm volatile("" ::: "memory");
  return old;
}

template <int FMT, bool STATE_BF16, bool SCALE_BF16, int ALGO, int ROUND, int CP>
__global__ __launch_bounds__(RES_WAVES * 64, RES_WAVES / 4) void eco_step_resident_kernel(const StepArgs a) {
  constexpr bool ADAM = algo_is_adam(ALGO), MASTER = algo_is_master(ALGO);
  constexpr bool KEEP_D = ALGO == ALGO_ADAM;                       // the injection of the other variants does not use d
  // fp32 v~ is stored at once; a bf16 one, rounded, could not stand in for the exact value in a tile that is finished from
  // memory, so it waits with the rest
  constexpr bool KEEP_V = ADAM && STATE_BF16;
  constexpr int D = RES_DEPTH, WAVES = RES_WAVES;
  constexpr uint64_t SLAB = RES_SLAB;
  __shared__ float4 d_ring[KEEP_D ? D * WAVES * 128 : 1];          // [slot][wave][half of the 8 values][lane]
  __shared__ uint32_t part_max[RES_RING], part_count[RES_RING], event_max[4], event_count[4];
  if (threadIdx.x < RES_RING) { part_max[threadIdx.x] = 0; part_count[threadIdx.x] = 0; }
  if (threadIdx.x < 4) { event_max[threadIdx.x] = 0; event_count[threadIdx.x] = 0; }
  __syncthreads();

  const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t n = (a.num_slabs - blockIdx.x + a.resident_wgs - 1) / a.resident_wgs;      // slabs of this workgroup
  const auto slab_of = [&](uint32_t i) { return blockIdx.x + i * a.resident_wgs; };
  // element offset of the wave's tile in its tensor
  const auto tile_at = [&](const TensorDesc &td, uint32_t slab) { return ((uint64_t)(slab - td.first_unit) * WAVES + wave) * TILE_ELEMS; };
  const auto tensor_of = [&](uint32_t i) { return load_table(a.slab_tensor, slab_of(i < n ? i : n - 1)); };

  // in hand: theta~ and m~ of D tiles (d beside them in LDS), and the tensors of their slabs
  float th[D][8], m[D][8];
  eco_u32x4_t v_kept[KEEP_V ? D : 1];
  uint32_t ti[D];
  // elements of the wave's tile at `tile` of a tensor (none beyond its end)
  const auto len_at = [&](uint64_t tile, uint64_t numel) {
    return (uint32_t)(tile >= numel ? 0 : numel - tile < TILE_ELEMS ? numel - tile : TILE_ELEMS);
  };
  // of the slab whose loads are under way: what they bring, where fp32 v~ goes, the place and length of the wave's tile
  RawLane<FMT, STATE_BF16, ALGO> raw;
  void *next_v;
  uint64_t next_tile;
  uint32_t next_len;
  uint32_t ti_next = tensor_of(0), ti_after = tensor_of(1);        // tensors of that slab and of the one after it
  const auto start_loads = [&](const TensorDesc &td, uint32_t slab, bool any) {
    next_tile = tile_at(td, slab);
    next_len = any ? len_at(next_tile, td.numel) : 0;
    next_v = td.v;
    load_raw<FMT, STATE_BF16, SCALE_BF16, ALGO, CP>(td, next_tile, next_len, lane, raw);
  };
  start_loads(load_tensor_desc(a, ti_next), slab_of(0), true);

  uint32_t known_ti = 0xFFFFFFFFu, known = NO_MAX, events = 0, tries = a.resident_tries;
  uint32_t entry = 0;                                              // one of slab_max[]'s entries of a tensor (or 0)
  bool wanted = false;                                             // this turn's finish needs an event
  // A wave's part in an event: the maximum of its share of the entries, or that one is missing.
  const auto contribute = [&](uint32_t x) {
    if (lane == 0) {
      lds_max(&event_max[events & 3], x);
      if (lds_add1(&event_count[events & 3]) == (events >> 2) * WAVES + WAVES - 1)
        lds_write(&event_max[(events + 2) & 3], 0u);               // all waves have left the events before this one
    }
  };
  const auto slabs_in = [&](const TensorDesc &td) { return td.numel <= SLAB ? 1u : (uint32_t)((td.numel + SLAB - 1) / SLAB); };

  for (uint32_t base = 0; base < n + D - 1; base += D) {
#pragma unroll
    for (int s = 0; s < D; ++s) {
      const uint32_t i = base + s;
      const int o = (s + 1) % D;                                   // the oldest slab in hand once slab i is
      const bool begin = i < n, finish = i + 1 >= D && i + 1 - D < n;
      const uint64_t tile = next_tile;
      const uint32_t len = next_len;                               // 0 unless begin
      void *const v_out = next_v;
      float g[8], v[8], w[8], x[8], d[8], sc = 1.0f;

      // theta~ of the wave's tile of slab i
      const TensorDesc tn = load_tensor_desc(a, ti_after);         // for the next loads
      ti[s] = ti_next;
      const eco_u32x4_t graw[2] = {raw.g, raw.g};
      unpack8<true>(graw, g);
      unpack_tile<STATE_BF16, CP>(raw.m, m[s]);
      if (ADAM) unpack_tile<STATE_BF16, CP>(raw.v, v);
      if (MASTER) {
        unpack_tile<false, CP>(raw.w, w);
      } else {
        sc = decode8<FMT>(raw.c, raw.s, w);
        if (!exact_scale<SCALE_BF16, ALGO>()) {
#pragma unroll
          for (int j = 0; j < 8; ++j) w[j] *= sc;
        }
      }
      moments_lane<ALGO>(a, g, m[s], v, x);
      ti_next = ti_after;
      start_loads(tn, slab_of(i + 1 < n ? i + 1 : n - 1), i + 1 < n);
      ti_after = tensor_of(i + 2);
      if (KEEP_V) v_kept[KEEP_V ? s : 0] = pack_bf16x8(v);
      else if (ADAM) store_f32_tile<CP>(tile_buffer(v_out, tile, len, 4), v);
      // the entries loaded at the end of the last turn, normally complete: half a turn before the sum of them is wanted
      const bool early = wanted && wave_all(entry != NO_MAX);
      if (early) contribute(wave_umax(entry));
      uint32_t arrived = 0;
      if (begin) {
        theta_lane<SCALE_BF16, ALGO, ACC_FULL>(a, x, w, sc, m[s], 8, d, th[s]);
        if (len < TILE_ELEMS) fill_missing<ACC_WHOLE>(th[s], lane * ELEMS_PER_LANE < len ? 8 : 0, 0.0f);
        if (KEEP_D) {
          float4 *p = d_ring + (s * WAVES + wave) * 128 + lane;
          p[0] = make_float4(d[0], d[1], d[2], d[3]);
          p[64] = make_float4(d[4], d[5], d[6], d[7]);
        }
        const uint32_t wmax = wave_umax(f2u(absmax8(th[s])));
        if (lane == 0) {
          lds_max(&part_max[i % RES_RING], wmax);
          arrived = lds_add1(&part_count[i % RES_RING]) + 1;       // looked at once the random words below are under way
        }
      }

      // the wave's tile of slab i - (D - 1)
      const uint32_t slab = slab_of(finish ? i + 1 - D : 0);
      const TensorDesc td = load_tensor_desc(a, finish ? ti[o] : ti_next);
      const uint64_t out = tile_at(td, slab);
      Philox4 r = {0, 0, 0, 0};
      // (the key schedule is derived from the seed anew each time: kept across the loop it takes 20 scalar registers)
      uint32_t seed_lo = a.seed_lo, seed_hi = a.seed_hi;
      asm volatile("" : "+s"(seed_lo), "+s"(seed_hi));
      if (finish) r = random_lane<ROUND>(a, td, out + lane * ELEMS_PER_LANE, seed_lo, seed_hi);

      // the workgroup's last wave at slab i publishes the slab's maximum
      const bool last = begin && arrived == (i / RES_RING + 1) * WAVES;            // in lane 0
      uint32_t slab_x = 0;
      if (last) {
        slab_x = lds_read(&part_max[i % RES_RING]);
        lds_write(&part_max[i % RES_RING], 0u);
        const TensorDesc tl = load_tensor_desc(a, ti[s]);
        if (tl.slot && (uint64_t)(slab_of(i) + 1 - tl.first_unit) * SLAB >= tl.numel) {      // its last slab, and it has a tail
          const uint32_t y = a.tail_max[tl.group_size];
          slab_x = slab_x > y ? slab_x : y;
        }
      }
      __builtin_amdgcn_raw_buffer_store_b32(slab_x, __builtin_amdgcn_make_buffer_rsrc(a.slab_max + slab_of(begin ? i : 0), 0, 4, 0x00020000),
                                            last ? 0 : 4, 0, SCOPE_AGENT);

      uint32_t out_len = 0, cn[2] = {0, 0};
      float eo[8] = {};
      if (finish) {
        if (ti[o] != known_ti || known == NO_MAX) {
          if (!early) {
            bool all = false;
            for (uint32_t t = 0; !all && t < tries; ++t) {
              entry = threadIdx.x < slabs_in(td) ? __hip_atomic_load(a.slab_max + td.first_unit + threadIdx.x, __ATOMIC_RELAXED,
                                                                     __HIP_MEMORY_SCOPE_AGENT) : 0u;
              all = wave_all(entry != NO_MAX);
              if (!all) __builtin_amdgcn_s_sleep(8);
            }
            contribute(all ? wave_umax(entry) : NO_MAX);
          }
          const uint32_t q = events & 3, full = (events >> 2) * WAVES + WAVES;
          while (lds_read(&event_count[q]) < full) __builtin_amdgcn_s_sleep(1);
          asm volatile("" ::: "memory");
          known = __builtin_amdgcn_readfirstlane(lds_read(&event_max[q]));
          known_ti = ti[o];
          ++events;
          if (known == NO_MAX) tries = 0;          // the others are not running: do not wait for them again
        }
        out_len = len_at(out, td.numel);
        if (known == NO_MAX) {
          if (threadIdx.x == 0) a.deferred[slab] = a.resident_counts[0] = 1;
          out_len = 0;
        }
      }
      if (ALGO == ALGO_SGDM_EXACT) {
        eco_u32x4_t q[2];
        load_f32_tile<CP>(tile_buffer(td.aux, out, out_len, 4), q);
        unpack_tile<false, CP>(q, eo);
      }
      if (out_len) {
        if (KEEP_D) {
          const float4 *p = d_ring + (o * WAVES + wave) * 128 + lane;
          const float4 lo = p[0], hi = p[64];
          d[0] = lo.x; d[1] = lo.y; d[2] = lo.z; d[3] = lo.w; d[4] = hi.x; d[5] = hi.y; d[6] = hi.z; d[7] = hi.w;
        }
        float qn[8];
        const int nvalid = lane * ELEMS_PER_LANE < out_len ? 8 : 0;
        const float s_new = quantize_lane8<FMT, SCALE_BF16, ROUND, ACC_WHOLE>(u2f(known), r, nvalid, th[o], cn, qn);
        if (!MASTER) inject_lane8<SCALE_BF16, ALGO>(a, s_new, th[o], qn, d, m[o], eo);
      }
      if (FMT == FMT_FP8)
        __builtin_amdgcn_raw_buffer_store_b64(eco_u32x2_t{cn[0], cn[1]}, tile_buffer(td.w, out, out_len, 1), lane * 8, 0, CP);
      else
        __builtin_amdgcn_raw_buffer_store_b32(cn[0], tile_buffer(td.w, out >> 1, out_len >> 1, 1), lane * 4, 0, CP);
      if (MASTER) store_f32_tile<CP>(tile_buffer(td.aux, out, out_len, 4), th[o]);
      if (ALGO == ALGO_SGDM_EXACT) store_f32_tile<CP>(tile_buffer(td.aux, out, out_len, 4), eo);
      store_state_tile<STATE_BF16, CP>(td.m, out, out_len, lane, m[o]);
      if (KEEP_V) store16<CP>(tile_buffer(td.v, out, out_len, 2), lane * 16, v_kept[KEEP_V ? o : 0]);

      // the entries the next turn's event wants, if there is one
      const uint32_t t = ti[(s + 2) % D];
      wanted = i + 2 >= D && i + 2 - D < n && (t != known_ti || known == NO_MAX);
      const TensorDesc te = load_tensor_desc(a, wanted ? t : ti_next);
      entry = __builtin_amdgcn_raw_buffer_load_b32(
          __builtin_amdgcn_make_buffer_rsrc(a.slab_max + te.first_unit, 0, wanted ? (int)(slabs_in(te) * 4) : 0, 0x00020000),
          threadIdx.x * 4, 0, SCOPE_AGENT | (int)0x80000000);
    }
  }
}

// The tail of a tensor, its last numel % 8 elements, is not in the slabs.  This kernel leaves the maximum of theta~ over it
// for the workgroup that publishes the tensor's last slab; the finishing kernel steps it.  A wave to each tensor.
template <int FMT, bool STATE_BF16, bool SCALE_BF16, int ALGO, int ROUND>
__global__ __launch_bounds__(RES_FINISH_THREADS) void eco_step_resident_tail_kernel(const StepArgs a) {
  const uint32_t x = a.unit_base + blockIdx.x * (RES_FINISH_THREADS / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (x >= a.num_resident) return;
  const TensorDesc td = load_tensor_desc(a, load_table(a.resident_tensor, x));
  if (!td.slot) return;
  step_lane<FMT, STATE_BF16, SCALE_BF16, ALGO, ROUND, ACC_GUARDED, RED_TILE>(a, td, td.numel, (threadIdx.x & 63) ? 0 : (int)td.slot, 0, false,
                                                                             a.tail_max + x);
}

// Finishes the slabs that were marked, from memory (normally none), a workgroup to each; then writes the tensors' new
// scales and empties their entries of slab_max[], a wave to each tensor.  Where slabs were marked, the last workgroup
// through with them does that alone: until then the old scales are needed.
template <int FMT, bool STATE_BF16, bool SCALE_BF16, int ALGO, int ROUND>
__global__ __launch_bounds__(RES_FINISH_THREADS) void eco_step_resident_finish_kernel(const StepArgs a) {
  constexpr uint32_t WAVES = RES_WAVES, NW = RES_FINISH_THREADS / 64;
  constexpr uint64_t SLAB = RES_SLAB;
  const uint32_t lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint32_t marked = __builtin_amdgcn_readfirstlane(a.resident_counts[0]);
  const auto slabs_of = [&](const TensorDesc &td) { return td.numel <= SLAB ? 1u : (uint32_t)((td.numel + SLAB - 1) / SLAB); };
  const auto max_of = [&](const TensorDesc &td) {
    uint32_t x = 0;
    for (uint32_t k = lane; k < slabs_of(td); k += 64) { const uint32_t y = a.slab_max[td.first_unit + k]; x = x > y ? x : y; }
    return wave_umax(x);
  };
  uint32_t first = blockIdx.x * NW + wave, stride = a.resident_wgs * NW;
  if (marked) {
    for (uint32_t slab = blockIdx.x; slab < a.num_slabs; slab += a.resident_wgs) {
      if (!__builtin_amdgcn_readfirstlane(a.deferred[slab])) continue;
      const TensorDesc td = load_tensor_desc(a, load_table(a.slab_tensor, slab));
      uint32_t amax = max_of(td);
      for (uint32_t k = wave; k < WAVES; k += NW) {
        const uint64_t e0 = ((uint64_t)(slab - td.first_unit) * WAVES + k) * TILE_ELEMS + lane * ELEMS_PER_LANE;
        step_lane<FMT, STATE_BF16, SCALE_BF16, ALGO, ROUND, ACC_WHOLE, RED_SLOT, CACHED, !STATE_BF16>(a, td, e0, e0 < td.numel ? 8 : 0, 0, false, &amax);
      }
    }
    __shared__ uint32_t last;
    __syncthreads();
    if (threadIdx.x == 0) last = atomicAdd(&a.resident_counts[1], 1u) == a.resident_wgs - 1;
    __syncthreads();
    if (!last) return;
    if (threadIdx.x < 2) a.resident_counts[threadIdx.x] = 0;
    for (uint32_t i = threadIdx.x; i < a.num_slabs; i += RES_FINISH_THREADS) a.deferred[i] = 0;
    first = wave;
    stride = NW;
  }
  for (uint32_t x = first; x < a.num_resident; x += stride) {
    const TensorDesc td = load_tensor_desc(a, load_table(a.resident_tensor, x));
    uint32_t amax = max_of(td);
    if (td.slot)
      step_lane<FMT, STATE_BF16, SCALE_BF16, ALGO, ROUND, ACC_GUARDED, RED_SLOT>(a, td, td.numel, lane ? 0 : (int)td.slot, 0, false, &amax);
    float s_new, inv;
    block_scale<FMT, SCALE_BF16>(u2f(amax), s_new, inv);
    if (lane == 0) store_scale<SCALE_BF16>(td, 0, s_new);
    for (uint32_t k = lane; k < slabs_of(td); k += 64) a.slab_max[td.first_unit + k] = NO_MAX;
  }
}

template <int FMT, bool STATE_BF16, bool SC, int RD, int AL>
hipError_t launch_resident(const StepLaunch &sl, hipStream_t stream) {
  const unsigned block = RES_WAVES * 64;
  const uint64_t fit = sl.max_launch_threads / block;
  const unsigned most = fit < 1 ? 1 : fit > 65536 ? 65536 : static_cast<unsigned>(fit);
  unsigned wgs = sl.resident_wgs < sl.args.num_slabs ? sl.resident_wgs : sl.args.num_slabs;
  if (wgs > most) wgs = most;
  const unsigned per_tensor = (sl.args.num_resident + RES_FINISH_THREADS / 64 - 1) / (RES_FINISH_THREADS / 64);
  StepArgs ta = sl.args;
  for (unsigned done = 0; sl.args.resident_tails && done < per_tensor; done += 2 * most) {
    ta.unit_base = done * (RES_FINISH_THREADS / 64);
    ECO_LAUNCH_CHECKED((eco_step_resident_tail_kernel<FMT, STATE_BF16, SC, AL, RD>), dim3(per_tensor - done < 2 * most ? per_tensor - done : 2 * most),
                       dim3(RES_FINISH_THREADS), 0, stream, ta);
  }
  ta = sl.args;
  ta.resident_wgs = wgs;
  if (sl.stream >> STREAM_TENSORWISE & 1u)
    ECO_LAUNCH_CHECKED((eco_step_resident_kernel<FMT, STATE_BF16, SC, AL, RD, STREAM_WAVE>), dim3(wgs), dim3(block), 0, stream, ta);
  else
    ECO_LAUNCH_CHECKED((eco_step_resident_kernel<FMT, STATE_BF16, SC, AL, RD, CACHED>), dim3(wgs), dim3(block), 0, stream, ta);
  unsigned fin = res_finish_workgroups(sl.args.num_resident, sl.args.num_slabs, sl.resident_wgs);
  if (fin > 2 * most) fin = 2 * most;
  ta.resident_wgs = fin;
  ECO_LAUNCH_CHECKED((eco_step_resident_finish_kernel<FMT, STATE_BF16, SC, AL, RD>), dim3(fin), dim3(RES_FINISH_THREADS), 0, stream, ta);
  return hipSuccess;
}

}  // namespace eco
