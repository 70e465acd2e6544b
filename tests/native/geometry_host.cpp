// Host-only checks of the launch geometry the library derives from a tensor's scale group: which class of kernel
// steps it, how many rows a workgroup of the wide-group kernel takes, and what one helper launch can hold.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "eco_internal.hpp"

#define CHECK(c)                                                   \
  do {                                                             \
    if (!(c)) { std::printf("FAILED line %d: %s\n", __LINE__, #c); return 1; } \
  } while (0)

int main() {
  using namespace eco;
  // classes
  CHECK(classify_group(128, 1 << 20) == GROUP_BLOCK && classify_group(32, 100) == GROUP_BLOCK && classify_group(512, 7) == GROUP_BLOCK);
  CHECK(classify_group(1024, 1 << 20) == GROUP_WIDE && classify_group(8192, 1 << 20) == GROUP_WIDE && classify_group(24, 1 << 20) == GROUP_WIDE);
  CHECK(classify_group(1000, 1 << 20) == GROUP_WIDE && classify_group(1 << 20, 4096) == GROUP_WIDE);       // one scale, small tensor
  CHECK(classify_group(1 << 20, 1 << 20) == GROUP_TENSOR && classify_group(8200, 8200) == GROUP_TENSOR && classify_group(1 << 30, 100) == GROUP_TENSOR);
  CHECK(classify_group(8200, 1 << 20) == GROUP_UNSUPPORTED && classify_group(20, 1 << 20) == GROUP_UNSUPPORTED && classify_group(16, 1 << 20) == GROUP_WIDE);

  // rows to a workgroup: known cases
  struct { uint64_t rows_in_tensor, g; uint32_t rows, waves; } known[] = {
      {2304, 576, 8, 9}, {576, 2304, 2, 9}, {2048, 1408, 4, 11}, {64, 640, 4, 5}, {6, 768, 2, 3}, {8, 1152, 4, 9},
      {5, 1408, 1, 3},          // not a whole number of bundles
      {4, 1024, 1, 2}, {4, 2048, 1, 4}, {3, 8192, 1, 16}, {16, 1000, 1, 2}, {8, 520, 1, 2}, {2, 6912, 1, 14}, {64, 96, 1, 1},
      {2, 7936, 1, 16},         // two rows would need 31 waves
  };
  for (const auto &k : known) {
    const WideGeometry w = wide_geometry(k.rows_in_tensor * k.g, k.g);
    if (w.rows != k.rows || w.waves != k.waves || w.units != k.rows_in_tensor / k.rows) {
      std::printf("FAILED: %llu rows of %llu: got %u rows, %u waves, %llu units\n", (unsigned long long)k.rows_in_tensor,
                  (unsigned long long)k.g, w.rows, w.waves, (unsigned long long)w.units);
      return 1;
    }
  }
  // a ragged last row never bundles
  CHECK(wide_geometry(8 * 1408 + 8, 1408).rows == 1 && wide_geometry(8 * 1408 + 8, 1408).units == 9);
  // every group length and a few row counts: what the kernel relies on
  for (uint64_t g = 8; g <= MAX_WIDE_GROUP; g += 8) {
    for (uint64_t n : {1ull, 2ull, 3ull, 4ull, 7ull, 8ull, 16ull, 24ull, 1000ull}) {
      const WideGeometry w = wide_geometry(n * g, g);
      CHECK(w.waves >= 1 && w.waves <= (uint32_t)MAX_WIDE_WAVES && w.rows >= 1 && w.rows <= 8);
      CHECK(w.units * w.rows == n);
      if (w.rows == 1) {
        CHECK(w.waves == (g + TILE_ELEMS - 1) / TILE_ELEMS);
      } else {
        CHECK(g > (uint64_t)TILE_ELEMS && (uint64_t)w.rows * g == (uint64_t)w.waves * TILE_ELEMS);   // every lane busy, whole rows
        CHECK(2 * g > (uint64_t)TILE_ELEMS);                                                          // a wave meets at most two rows
      }
    }
  }
  // what one helper launch holds
  CHECK(flat_call_fits((1ull << 35) - 512, 128) && !flat_call_fits(1ull << 35, 128) && !flat_call_fits((1ull << 40) + 1, 128));
  CHECK(flat_call_fits(1ull << 34, 520) && !flat_call_fits(1ull << 35, 520) && flat_call_fits(1ull << 30, 1ull << 31));
  // the helper kernels with more than 64 threads to a workgroup, up to the largest call: every launch within the limit,
  // together the whole array
  for (uint64_t n : {1ull, 2048ull, 2049ull, (1ull << 35) - 2048, (1ull << 35) - 2047, (1ull << 35) - 1024, (1ull << 35) - 1023, (1ull << 35) - 512}) {
    for (unsigned threads : {64u, 128u, 256u}) {
      CHECK(flat_call_fits(n, n) && flat_call_fits(n, 128));
      const FlatLaunch f = flat_launch(n, threads);
      uint64_t covered = 0;
      for (uint64_t first = 0; first < f.workgroups; first += f.per_launch) {
        const uint64_t k = f.workgroups - first < f.per_launch ? f.workgroups - first : f.per_launch;
        CHECK(k >= 1 && k * threads <= MAX_LAUNCH_THREADS && first <= 0xFFFFFFFFull);
        covered += k;
      }
      CHECK(covered == f.workgroups && covered * threads * ELEMS_PER_LANE >= n && (covered - 1) * threads * ELEMS_PER_LANE < n);
    }
  }
  // the second tensor-wise pass: every tile once, on the XCD of the first pass (workgroups go to eight in turn), the last ones first
  for (uint32_t n : {1u, 7u, 8u, 9u, 15u, 16u, 17u, 4099u}) {
    std::vector<bool> seen(n, false);
    for (uint32_t i = 0; i < n; ++i) {
      const uint32_t u = backwards_on_the_same_xcd(i, n);
      CHECK(u < n && !seen[u] && u % 8 == i % 8);
      CHECK(i < 8 || i >= n / 8 * 8 || backwards_on_the_same_xcd(i - 8, n) == u + 8);
      seen[u] = true;
    }
  }
  // the finishing kernel of the one-pass tensor-wise step has enough workgroups for every slab it may be left with
  for (unsigned cus : {32u, 256u}) {
    for (uint64_t slabs : {1ull, 21ull, 768ull, 15360ull, 1000000ull}) {
      for (uint64_t tensors : {1ull, 3ull, 1000ull, 100000ull}) {
        const unsigned wgs = res_finish_workgroups(tensors, slabs, cus);
        CHECK(wgs >= 1 && wgs <= 4 * cus && wgs >= (slabs < cus ? slabs : cus));
        CHECK(slabs > tensors || static_cast<uint64_t>(wgs) * 4 >= tensors || wgs == 4 * cus);
      }
    }
  }
  // an LDS request that the hardware's LDS holds k times, and none where k is no less than the waves of a compute unit
  for (unsigned k = 0; k <= 2000; ++k) {
    const uint32_t lds = lds_for_workgroups(k);
    CHECK(k == 0 || k >= 32 ? lds == 0 : lds > 0 && lds <= 65536 && (lds + 128 + 1279) / 1280 * 1280 * k <= 163840);
    if (k > 2 && k < 32) CHECK((lds + 1279) / 1280 * 1280 * (k + k / 4 + 1) > 163840);
  }
  // how many workgroups are to be resident, 0 for no wish.  Full rows: at least two, at least 20 waves where bf16 state is capped.
  // Rows with idle lanes, and units of one wave: the fewest with a certain number of waves' worth of busy lanes, whatever their share
  for (int algo : {ALGO_ADAM, ALGO_SGDM, ALGO_SGDM_EXACT, ALGO_ADAM_MASTER, ALGO_SGDM_MASTER}) {
    for (int bf16 = 0; bf16 <= 1; ++bf16) {
      const KernelVariant kv = {FMT_FP8, bf16, bf16, algo, ROUND_SR};
      for (unsigned nw = 2; nw <= (unsigned)MAX_WIDE_WAVES; ++nw) {
        const unsigned k = wide_workgroups(kv, nw);
        CHECK(k == 0 || (k >= 2 && k * nw <= 32));
        if (algo == ALGO_ADAM && bf16) CHECK(k == 0 || (k * nw >= 20 && (nw <= 4 || nw == 8)));
      }
      for (uint64_t g = 520; g < MAX_WIDE_GROUP; g += 8) {
        if (g % TILE_ELEMS == 0) continue;
        const uint64_t nw = (g + TILE_ELEMS - 1) / TILE_ELEMS;
        const bool nearly_all = (nw <= 4 || nw == 8) && g * 20 >= nw * TILE_ELEMS * 19;
        for (uint64_t mb : {100ull, 599ull, 600ull, 5000ull}) {
          const bool capped = algo == ALGO_ADAM          ? !bf16 || (mb >= 600 && nearly_all)
                              : algo == ALGO_ADAM_MASTER ? bf16 || mb >= 600
                                                         : !(algo == ALGO_SGDM && bf16);
          const unsigned k = wide_workgroups_idle(kv, mb * 1000000, (unsigned)nw, 1000, 1000 * g);
          const unsigned half = wide_workgroups_idle(kv, mb * 1000000, (unsigned)nw, 1000, 500 * g);
          CHECK(capped ? k >= 2 && k <= 22 : k == 0);
          CHECK(half == 0 || (half >= k && half <= 2 * k));
          if (k > 2) CHECK(k * g * 10 >= 85 * TILE_ELEMS && (k - 1) * g * 10 < 204 * TILE_ELEMS && k * nw <= 44);
        }
      }
      for (uint64_t busy = 1; busy <= (uint64_t)TILE_ELEMS; ++busy) {
        for (uint64_t mb : {1ull, 100ull, 191ull, 192ull, 383ull, 384ull, 767ull, 768ull, 5000ull}) {
          const unsigned k = unit_workgroups(kv, mb * 1000000, 1000, 1000 * busy);
          CHECK(k == 0 || (k * busy * 10 >= 70 * TILE_ELEMS && (k - 1) * busy * 10 < 215 * TILE_ELEMS));
          CHECK(k == 0 || mb >= 384 || (!bf16 && (algo == ALGO_ADAM || (algo == ALGO_ADAM_MASTER && mb >= 192))));
          CHECK(lds_for_workgroups(k) == 0 || (k < 32 && (lds_for_workgroups(k) + 1279) / 1280 * 1280 * k <= 163840));
        }
      }
    }
  }
  // the step's own grouping of rows, every group length, a ragged last row among the numbers of rows: what the kernels rely on.  At
  // most 16 groups in a workgroup's LDS, also where a list launch packs several units into one of any number of waves; a wave meets at
  // most two groups; units of Adam with master weights of several rows have no idle lane, in the last workgroup neither
  for (int opt = 0; opt < 8; ++opt) {
    const StateLayout l = {(opt & 1) != 0, (opt & 2) != 0, (opt & 4) != 0};
    for (uint64_t g = 520; g <= MAX_WIDE_GROUP; g += 8) {
      for (uint64_t n : {1ull, 2ull, 3ull, 4ull, 5ull, 7ull, 8ull, 15ull, 16ull, 24ull, 1000ull}) {
        for (uint64_t cut : {0ull, 8ull, 3ull, 515ull}) {
          const uint64_t numel = n * g - cut;
          const WideGeometry w = step_geometry(numel, g < numel ? g : numel, l);
          const uint64_t group = g < numel ? g : numel, groups = (numel + group - 1) / group;
          CHECK(w.rows >= 1 && w.rows <= 8 && w.waves >= 1 && w.waves <= (uint32_t)MAX_WIDE_WAVES);
          CHECK(w.waves == (w.rows * group + TILE_ELEMS - 1) / TILE_ELEMS && w.rows <= groups);
          CHECK(w.units * w.rows >= groups && (w.units - 1) * w.rows < groups);
          if (w.rows > 1) CHECK(group > (uint64_t)TILE_ELEMS);
          for (uint32_t nw = w.waves; nw <= (uint32_t)MAX_WIDE_WAVES; ++nw) CHECK(nw / w.waves * w.rows <= 16);
          if (l.aux && l.adam && w.rows > 1) CHECK(w.rows * group == (uint64_t)w.waves * TILE_ELEMS && w.units * w.rows * group == numel);
          const StepRows rows = {l, true};
          const Placement p = place_tensor(numel, g, GROUP_WIDE, true, FMT_FP8, TILE_ELEMS, 0, &rows);
          if (group > (uint64_t)TILE_ELEMS) {
            CHECK(p.kind == UNIT_WIDE && p.list == LIST_WIDE1 + (int)w.waves - 1 && p.units == w.units && p.rows == w.rows);
            CHECK(p.entries == wide_geometry(numel, group).units && p.idle == (w.rows * group % TILE_ELEMS != 0));
          }
        }
      }
    }
  }
  struct { uint64_t n, g; bool adam, bf16, aux; uint32_t rows, waves; } own[] = {
      {2304, 576, true, false, false, 8, 9}, {1001, 576, true, false, false, 3, 4}, {2, 576, true, false, false, 2, 3}, {1000, 1152, true, false, false, 2, 5},
      {1000, 1152, true, true, false, 4, 9}, {2048, 1408, true, false, false, 1, 3}, {2048, 1408, true, true, false, 4, 11},
      {2048, 1408, true, false, true, 4, 11}, {1001, 896, false, false, false, 4, 7}, {1001, 760, true, false, false, 2, 3}, {1001, 1000, true, false, false, 1, 2},
      {1001, 1152, false, false, true, 2, 5}, {1001, 1152, true, false, true, 1, 3}};
  for (const auto &k : own) {
    const WideGeometry w = step_geometry(k.n * k.g, k.g, {k.adam, k.bf16, k.aux});
    if (w.rows != k.rows || w.waves != k.waves) {
      std::printf("FAILED: step, %llu rows of %llu: got %u rows, %u waves\n", (unsigned long long)k.n, (unsigned long long)k.g, w.rows, w.waves);
      return 1;
    }
  }
  CHECK(place_tensor(64 * 1000, 1000, GROUP_WIDE, true, FMT_FP8).idle && place_tensor(3 * 1408, 1408, GROUP_WIDE, true, FMT_FP8).idle);
  CHECK(!place_tensor(4 * 1408, 1408, GROUP_WIDE, true, FMT_FP8).idle && !place_tensor(5 * 1024, 1024, GROUP_WIDE, true, FMT_FP8).idle);
  // tensor-wise scaling: one pass where it was measured to pay, and more readily with fewer launches in its way
  for (int opt = 0; opt < 16; ++opt) {
    const StateLayout l = {(opt & 1) != 0, (opt & 2) != 0, (opt & 4) != 0, (opt & 8) != 0};
    CHECK(one_pass_pays(l, 1, 1, 256, false, false) && one_pass_pays(l, 1, 256, 256, false, false));
    CHECK(!one_pass_pays(l, 17000000, 257, 256, false, false) && !one_pass_pays(l, 1, 1, 256, true, false) && !one_pass_pays(l, 1, 1, 256, false, true));
    bool before[4] = {false, false, false, false};
    for (uint64_t bytes = 1 << 20; bytes < 1ull << 31; bytes += bytes / 8) {
      for (int k = 0; k < 4; ++k) {
        const bool now = one_pass_pays(l, bytes, 1000, 256, (k & 1) != 0, (k & 2) != 0);
        CHECK(now || !before[k]);
        CHECK(!now || ((!(k & 1) || before[k - 1] || one_pass_pays(l, bytes, 1000, 256, false, (k & 2) != 0)) &&
                       (!(k & 2) || one_pass_pays(l, bytes, 1000, 256, (k & 1) != 0, false))));
        before[k] = now;
      }
    }
    CHECK(before[0] && before[1] && before[2] && before[3]);
  }
  CHECK(array_bytes(1000, FMT_FP8, {true, false, false}) == 11000 && array_bytes(1000, FMT_INT4, {true, true, false}) == 6500);
  CHECK(array_bytes(1000, FMT_FP8, {false, false, true}) == 11000 && array_bytes(1000, FMT_BF16_PLAIN, {true, true, true}) == 8000);
  // rows that the quantizer bundles, and rows that it leaves alone though the step bundles them
  for (uint64_t g : {576ull, 640ull, 768ull, 1152ull, 1280ull, 1792ull, 2304ull, 2816ull, 3840ull}) {
    const WideGeometry w = wide_geometry(64 * g, g);
    CHECK(w.rows > 1 && quantizer_takes_bundle(w.rows, g, FMT_FP8) && quantizer_takes_bundle(w.rows, g, FMT_INT4));
  }
  for (uint64_t g : {1408ull, 1920ull}) CHECK(!quantizer_takes_bundle(4, g, FMT_FP8) && !quantizer_takes_bundle(4, g, FMT_INT4));
  CHECK(quantizer_takes_bundle(4, 1664, FMT_FP8) && !quantizer_takes_bundle(4, 1664, FMT_INT4) && !quantizer_takes_bundle(4, 896, FMT_INT4));
  for (uint64_t g = 520; g <= MAX_WIDE_GROUP; g += 8) CHECK(!quantizer_takes_bundle(1, g, FMT_FP8) && !quantizer_takes_bundle(1, g, FMT_INT4));
  std::printf("geometry ok\n");
  return 0;
}
