/* What a step launches, without a GPU: this program's runtime calls stand before HIP's, record every launch and let it pass.
 * Each case says how many launches a plan's step makes and which of them ask for LDS, the request that caps resident waves. */
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <hip/hip_runtime_api.h>

#include "eco.h"

enum { MOST = 64 };
static int launches;
static size_t lds_of[MOST], pushed_lds;
static unsigned grid_of[MOST], block_of[MOST], pushed_grid, pushed_block;
static const void *kernel_of[MOST];

hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t stream) {
  (void)grid; (void)block; (void)args; (void)stream;
  if (launches < MOST) { kernel_of[launches] = f; lds_of[launches] = lds; grid_of[launches] = pushed_grid; block_of[launches] = pushed_block; }
  ++launches;
  return hipSuccess;
}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
  (void)stream;
  pushed_lds = lds; pushed_grid = grid.x; pushed_block = block.x;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *stream) {
  grid->x = grid->y = grid->z = block->x = block->y = block->z = 1;
  *lds = pushed_lds;
  *stream = NULL;
  return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGetDevice(int *device) { *device = 0; return hipSuccess; }
hipError_t hipSetDevice(int device) { (void)device; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *x, hipDeviceAttribute_t a, int device) { (void)a; (void)device; *x = 256; return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) { *p = malloc(n); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind k) { (void)k; memcpy(d, s, n); return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *symbol) { (void)symbol; *p = (void *)0x100000; return hipSuccess; }

enum { ROW = -1, TENSOR = -2, PLAIN = -3 };
enum { FP8 = ECO_FMT_FP8_E4M3, INT4 = ECO_FMT_INT4, F32 = ECO_DT_FP32, BF16 = ECO_DT_BF16, ADAM = ECO_OPT_ADAM, SGDM = ECO_OPT_SGDM };
typedef struct {
  const char *what;
  int fmt, state, opt, mode;
  struct { int count, scale; uint64_t rows, cols; } t[3];    /* scale: elements, or ROW, TENSOR, PLAIN */
  int launches;
  int capped;                                                /* bit i: launch i asks for LDS */
} Case;

static const Case cases[] = {
    /* full tiles: caps for arrays beyond the cache; Adam with fp32 state has one from 96 MB on.  (1 M elements, us, with a cap of 28 waves and
     * without: 5.25 and 5.27) */
    {"block bf16, 16 M", FP8, BF16, ADAM, ECO_MODE_ECO, {{16, 128, 1024, 1024}}, 1, 0},
    {"block bf16, 64 M", FP8, BF16, ADAM, ECO_MODE_ECO, {{64, 128, 1024, 1024}}, 1, 1},
    {"block bf16 INT4, 48 M", INT4, BF16, ADAM, ECO_MODE_ECO, {{48, 128, 1024, 1024}}, 1, 0},
    {"block bf16 INT4, 64 M", INT4, BF16, ADAM, ECO_MODE_NAIVE, {{64, 128, 1024, 1024}}, 1, 1},
    {"block bf16 master, 24 M", FP8, BF16, ADAM, ECO_MODE_MASTER, {{24, 128, 1024, 1024}}, 1, 0},
    {"block bf16 master, 48 M", FP8, BF16, ADAM, ECO_MODE_MASTER, {{48, 128, 1024, 1024}}, 1, 1},
    {"block fp32, 1 M", FP8, F32, ADAM, ECO_MODE_ECO, {{1, 128, 1024, 1024}}, 1, 0},
    {"block fp32, 10 M", FP8, F32, ADAM, ECO_MODE_ECO, {{10, 128, 1024, 1024}}, 1, 1},
    {"block bf16 SGDM", FP8, BF16, SGDM, ECO_MODE_ECO, {{128, 128, 1024, 1024}}, 1, 0},
    /* unquantized */
    {"plain, 4 M", FP8, F32, ADAM, ECO_MODE_ECO, {{4, PLAIN, 1024, 1024}}, 1, 0},
    {"plain, 16 M", FP8, F32, ADAM, ECO_MODE_ECO, {{16, PLAIN, 1024, 1024}}, 1, 1},
    {"plain bf16 SGDM, 48 M", FP8, BF16, SGDM, ECO_MODE_ECO, {{48, PLAIN, 1024, 1024}}, 1, 0},
    {"plain bf16 SGDM, 96 M", FP8, BF16, SGDM, ECO_MODE_ECO, {{96, PLAIN, 1024, 1024}}, 1, 1},
    /* rows; full ones that pass the caches by from 450 MB on (with caps of 28 waves and without: bf16 state of 768, 390 and 430 MB 97.5 and 97.1,
     * 116.8 and 116.2; master weights of 768, 110 MB 30.3 and 30.3) */
    {"rows of 768, bf16, 16 M", FP8, BF16, ADAM, ECO_MODE_ECO, {{20, ROW, 1024, 768}}, 1, 0},
    {"rows of 768, bf16, 63 M", FP8, BF16, ADAM, ECO_MODE_ECO, {{80, ROW, 1024, 768}}, 1, 0},
    {"rows of 768, bf16, 66 M", FP8, BF16, ADAM, ECO_MODE_ECO, {{84, ROW, 1024, 768}}, 1, 1},
    {"rows of 1000, bf16", FP8, BF16, ADAM, ECO_MODE_ECO, {{80, ROW, 1024, 1000}}, 1, 0},
    {"rows of 2304, bf16", FP8, BF16, ADAM, ECO_MODE_ECO, {{40, ROW, 1024, 2304}}, 1, 0},
    {"rows of 1000 and of 1024, bf16, a tenth idle", FP8, BF16, ADAM, ECO_MODE_ECO, {{9, ROW, 1024, 1000}, {81, ROW, 1024, 1024}}, 1, 1},
    {"rows of 1800, master", FP8, F32, ADAM, ECO_MODE_MASTER, {{20, ROW, 1024, 1800}}, 1, 0},
    {"rows of 768, master, 4 M", FP8, F32, ADAM, ECO_MODE_MASTER, {{5, ROW, 1024, 768}}, 1, 0},
    {"rows of 768, master, 8 M", FP8, F32, ADAM, ECO_MODE_MASTER, {{10, ROW, 1024, 768}}, 1, 0},
    {"rows of 768, master, 31 M", FP8, F32, ADAM, ECO_MODE_MASTER, {{40, ROW, 1024, 768}}, 1, 1},
    /* the step's own grouping of rows takes a launch more than the other only from 384 MB on */
    {"rows of 1024 and an odd number of 768, 110 MB", FP8, BF16, ADAM, ECO_MODE_ECO, {{10, ROW, 1024, 1024}, {10, ROW, 687, 768}}, 1, 0},
    {"rows of 1024 and an odd number of 768, 440 MB", FP8, BF16, ADAM, ECO_MODE_ECO, {{40, ROW, 1024, 1024}, {40, ROW, 687, 768}}, 2, 0},
    {"rows of 1024 and an odd number of 768, 480 MB", FP8, BF16, ADAM, ECO_MODE_ECO, {{44, ROW, 1024, 1024}, {44, ROW, 687, 768}}, 2, 3},
    {"rows of 2048 and an odd number of 576, 110 MB", FP8, BF16, ADAM, ECO_MODE_ECO, {{5, ROW, 1024, 2048}, {10, ROW, 915, 576}}, 1, 0},
    {"rows of 1000, 7 M, in the cache", FP8, F32, ADAM, ECO_MODE_ECO, {{7, ROW, 1024, 1000}}, 1, 0},
    {"rows of 1000, 10 M", FP8, F32, ADAM, ECO_MODE_ECO, {{10, ROW, 1024, 1000}}, 1, 1},
    {"rows of 1000, SGDM, 40 M", FP8, F32, SGDM, ECO_MODE_ECO, {{40, ROW, 1024, 1000}}, 1, 0},
    {"rows of 1000, SGDM, 60 M", FP8, F32, SGDM, ECO_MODE_ECO, {{60, ROW, 1024, 1000}}, 1, 1},
    {"rows of 1000, SGDM with a stored error, 30 M", FP8, F32, SGDM, ECO_MODE_EXACT, {{30, ROW, 1024, 1000}}, 1, 0},
    {"rows of 1000, SGDM with a stored error, 40 M", FP8, F32, SGDM, ECO_MODE_EXACT, {{40, ROW, 1024, 1000}}, 1, 1},
    {"rows of 1000, bf16 master, 40 M", FP8, BF16, ADAM, ECO_MODE_MASTER, {{40, ROW, 1024, 1000}}, 1, 1},
    {"rows of 1000, bf16 SGDM master, 40 M", INT4, BF16, SGDM, ECO_MODE_MASTER, {{40, ROW, 1024, 1000}}, 1, 0},
    {"rows of 1000, bf16 SGDM master, 50 M", INT4, BF16, SGDM, ECO_MODE_MASTER, {{50, ROW, 1024, 1000}}, 1, 1},
    {"rows of 1000, bf16 stored error, 50 M", INT4, BF16, SGDM, ECO_MODE_EXACT, {{50, ROW, 1024, 1000}}, 1, 1},
    {"rows of 1000, bf16 SGDM, 90 M", INT4, BF16, SGDM, ECO_MODE_ECO, {{90, ROW, 1024, 1000}}, 1, 0},
    {"rows of 1000, bf16, 90 M", FP8, BF16, ADAM, ECO_MODE_ECO, {{90, ROW, 1024, 1000}}, 1, 1},
    {"rows of 1800, bf16, 90 M, too few lanes busy", FP8, BF16, ADAM, ECO_MODE_ECO, {{50, ROW, 1024, 1800}}, 1, 0},
    {"rows of 1800, master, 44 M", FP8, F32, ADAM, ECO_MODE_MASTER, {{24, ROW, 1024, 1800}}, 1, 1},
    /* short rows: a launch of one-wave units alone has caps of its own, a few beside full tiles ride under theirs */
    {"rows of 400, SGDM, 57 M", FP8, F32, SGDM, ECO_MODE_ECO, {{140, ROW, 1024, 400}}, 1, 1},
    {"rows of 328, SGDM, 57 M, too few lanes busy", FP8, F32, SGDM, ECO_MODE_ECO, {{170, ROW, 1024, 328}}, 1, 0},
    {"rows of 400, 10 M, in part in the cache", FP8, F32, ADAM, ECO_MODE_ECO, {{25, ROW, 1024, 400}}, 1, 1},
    {"rows of 328, 10 M, in part in the cache", FP8, F32, ADAM, ECO_MODE_ECO, {{30, ROW, 1024, 328}}, 1, 0},
    {"rows of 328, 37 M", FP8, F32, ADAM, ECO_MODE_ECO, {{110, ROW, 1024, 328}}, 1, 1},
    {"rows of 504, bf16 INT4, 62 M", INT4, BF16, ADAM, ECO_MODE_ECO, {{120, ROW, 1024, 504}}, 1, 1},
    {"rows of 400, bf16 INT4, 62 M, too few lanes busy", INT4, BF16, ADAM, ECO_MODE_ECO, {{150, ROW, 1024, 400}}, 1, 0},
    {"rows of 400, SGDM", FP8, F32, SGDM, ECO_MODE_ECO, {{40, ROW, 1024, 400}}, 1, 0},
    {"rows of 160, master", FP8, F32, ADAM, ECO_MODE_MASTER, {{60, ROW, 1024, 160}}, 1, 0},
    {"rows of 160, master, 15 M", FP8, F32, ADAM, ECO_MODE_MASTER, {{94, ROW, 1024, 160}}, 1, 1},
    {"rows of 160, bf16 SGDM master, 30 M", FP8, BF16, SGDM, ECO_MODE_MASTER, {{190, ROW, 1024, 160}}, 1, 0},
    {"rows of 160, bf16 SGDM master, 50 M", FP8, BF16, SGDM, ECO_MODE_MASTER, {{310, ROW, 1024, 160}}, 1, 1},
    /* (off the lines of memory they have one however few lanes are busy: 50 M elements 159 us without, 147 with it) */
    {"rows of 328, bf16 SGDM master, 50 M", FP8, BF16, SGDM, ECO_MODE_MASTER, {{150, ROW, 1024, 328}}, 1, 1},
    {"rows of 264, bf16 master, 42 M", INT4, BF16, ADAM, ECO_MODE_MASTER, {{164, ROW, 1024, 264}}, 1, 1},
    {"rows of 320, bf16 master, 42 M, past the caches, too few lanes busy", INT4, BF16, ADAM, ECO_MODE_MASTER, {{135, ROW, 1024, 320}}, 1, 0},
    {"rows of 328, SGDM, 140 M", FP8, F32, SGDM, ECO_MODE_ECO, {{420, ROW, 1024, 328}}, 1, 1},
    {"rows of 328, INT4 SGDM, 140 M, too few lanes busy", INT4, F32, SGDM, ECO_MODE_ECO, {{420, ROW, 1024, 328}}, 1, 0},
    {"rows of 400, 5 M, in the cache", FP8, F32, ADAM, ECO_MODE_ECO, {{12, ROW, 1024, 400}}, 1, 0},
    {"rows of 160, bf16 stored error, 50 M", FP8, BF16, SGDM, ECO_MODE_EXACT, {{310, ROW, 1024, 160}}, 1, 1},
    {"rows of 504, bf16 SGDM, 120 M", FP8, BF16, SGDM, ECO_MODE_ECO, {{235, ROW, 1024, 504}}, 1, 0},
    {"rows of 504, bf16 SGDM, 170 M", FP8, BF16, SGDM, ECO_MODE_ECO, {{330, ROW, 1024, 504}}, 1, 1},
    {"a few rows of 400 beside blocks", FP8, F32, ADAM, ECO_MODE_ECO, {{60, 128, 1024, 1024}, {4, ROW, 1024, 400}}, 1, 1},
    /* one-wave units with few busy lanes beside arrays from HBM: as many waves as want to */
    {"100 norms of 32 beside a long one", FP8, F32, ADAM, ECO_MODE_ECO, {{1, TENSOR, 1, 70000000}, {100, PLAIN, 1, 32}}, 5, 10},
    {"100 tensors of 40 beside a long one", FP8, F32, ADAM, ECO_MODE_ECO, {{1, TENSOR, 1, 70000000}, {100, TENSOR, 1, 40}}, 5, 10},
    /* partial last tiles are one-wave units too, and count with the lanes they keep busy */
    {"tails and a few short rows beside a long one", FP8, F32, ADAM, ECO_MODE_ECO, {{1, TENSOR, 1, 70000000}, {1, ROW, 16, 400}, {1000, 128, 1, 500}}, 5, 11},
    /* tensor-wise: two launches in one pass (three with a tail), four in two passes, and which of these are capped */
    {"three small tensors", FP8, F32, ADAM, ECO_MODE_ECO, {{3, TENSOR, 1, 40000}}, 2, 0},
    {"three small tensors with tails", FP8, F32, ADAM, ECO_MODE_ECO, {{3, TENSOR, 1, 40001}}, 4, 5},
    {"two turns", INT4, BF16, ADAM, ECO_MODE_ECO, {{8, TENSOR, 1, 200000}}, 4, 0},
    {"many turns", INT4, BF16, ADAM, ECO_MODE_ECO, {{16, TENSOR, 1408, 2048}}, 2, 0},
    {"many turns with tails", INT4, BF16, ADAM, ECO_MODE_ECO, {{16, TENSOR, 1408, 2048}, {1, TENSOR, 1, 8193}}, 3, 0},
    /* ... and short ones of a length that is no multiple of 8: along with longer ones, unless a launch takes them for nothing */
    {"short odd ones beside longer ones", INT4, BF16, ADAM, ECO_MODE_ECO, {{2, TENSOR, 1, 11942}, {31, TENSOR, 1, 770}}, 4, 0},
    {"short odd ones beside one turn", INT4, BF16, ADAM, ECO_MODE_NAIVE, {{5, TENSOR, 18, 2048}, {29, TENSOR, 1, 2627}}, 4, 0},
    {"short odd ones beside longer ones and norms", INT4, BF16, ADAM, ECO_MODE_ECO, {{2, TENSOR, 1, 11942}, {31, TENSOR, 1, 770}, {1, PLAIN, 1, 512}}, 5, 0},
    {"short odd ones and norms beside one turn", INT4, BF16, ADAM, ECO_MODE_ECO, {{1, TENSOR, 1, 9000}, {31, TENSOR, 1, 770}, {1, PLAIN, 1, 512}}, 3, 0},
    {"short odd ones beside many turns", INT4, BF16, ADAM, ECO_MODE_ECO, {{16, TENSOR, 1408, 2048}, {29, TENSOR, 1, 2627}}, 3, 0},
    {"short odd ones beside many turns with tails", INT4, BF16, ADAM, ECO_MODE_ECO, {{16, TENSOR, 1408, 2048}, {1, TENSOR, 1, 8193}, {29, TENSOR, 1, 2627}}, 3, 0},
    {"many short odd ones beside a longer one", INT4, BF16, ADAM, ECO_MODE_ECO, {{1, TENSOR, 1, 9000}, {540, TENSOR, 1, 770}}, 3, 0},
    {"short odd ones alone", INT4, BF16, ADAM, ECO_MODE_ECO, {{31, TENSOR, 1, 770}}, 1, 0},
    /* ... either side of where one pass and two met, again with the second pass on the XCDs of the first */
    {"9.6 M, INT4 bf16", INT4, BF16, ADAM, ECO_MODE_ECO, {{32, TENSOR, 1, 300000}}, 4, 0},
    {"19 M, INT4 bf16", INT4, BF16, ADAM, ECO_MODE_ECO, {{64, TENSOR, 1, 300000}}, 2, 0},
    {"4.8 M, fp32", FP8, F32, ADAM, ECO_MODE_ECO, {{16, TENSOR, 1, 300000}}, 4, 5},
    {"7.2 M, fp32", FP8, F32, ADAM, ECO_MODE_ECO, {{24, TENSOR, 1, 300000}}, 2, 0},
    {"4.8 M, master", FP8, F32, ADAM, ECO_MODE_MASTER, {{16, TENSOR, 1, 300000}}, 4, 0},
    {"7.2 M, master", FP8, F32, ADAM, ECO_MODE_MASTER, {{24, TENSOR, 1, 300000}}, 2, 0},
    {"38 M with tails, master", FP8, F32, ADAM, ECO_MODE_MASTER, {{128, TENSOR, 1, 300001}}, 4, 0},
    {"38 M beside a long one, master", FP8, F32, ADAM, ECO_MODE_MASTER, {{128, TENSOR, 1, 300000}, {1, TENSOR, 1, 6000000}}, 4, 0},
    {"38 M beside a long one, SGDM, master", FP8, F32, SGDM, ECO_MODE_MASTER, {{128, TENSOR, 1, 300000}, {1, TENSOR, 1, 6000000}}, 4, 0},
    {"38 M beside a long one, stored error", FP8, F32, SGDM, ECO_MODE_EXACT, {{128, TENSOR, 1, 300000}, {1, TENSOR, 1, 6000000}}, 6, 0},
    /* ... and what makes one pass of a list with tails beside a longer tensor, by the kind of state */
    {"230 MB, SGDM", FP8, F32, SGDM, ECO_MODE_ECO, {{7, TENSOR, 1, 4700000}, {1, TENSOR, 1, 300007}, {1, TENSOR, 1, 5000000}}, 7, 0},
    {"420 MB", FP8, F32, ADAM, ECO_MODE_ECO, {{9, TENSOR, 1, 4700000}, {1, TENSOR, 1, 8193}, {1, TENSOR, 1, 6000000}}, 7, 40},
    {"420 MB, INT4 bf16", INT4, BF16, ADAM, ECO_MODE_ECO, {{14, TENSOR, 1, 4700000}, {1, TENSOR, 1, 8193}, {1, TENSOR, 1, 6000000}}, 7, 40},
    {"420 MB, SGDM INT4", INT4, F32, SGDM, ECO_MODE_ECO, {{14, TENSOR, 1, 4700000}, {1, TENSOR, 1, 8193}, {1, TENSOR, 1, 6000000}}, 7, 40},
    {"420 MB, stored error, bf16", FP8, BF16, SGDM, ECO_MODE_EXACT, {{10, TENSOR, 1, 4700000}, {1, TENSOR, 1, 8193}, {1, TENSOR, 1, 6000000}}, 7, 0},
    {"1.1 GB, master", FP8, F32, ADAM, ECO_MODE_MASTER, {{16, TENSOR, 1, 4700000}, {1, TENSOR, 1, 8193}, {1, TENSOR, 1, 6000000}}, 7, 0},
    {"1.1 GB, master INT4 bf16", INT4, BF16, ADAM, ECO_MODE_MASTER, {{23, TENSOR, 1, 4700000}, {1, TENSOR, 1, 8193}, {1, TENSOR, 1, 6000000}}, 7, 0},
    {"beside a long one", INT4, BF16, ADAM, ECO_MODE_ECO, {{8, TENSOR, 1, 870000}, {1, TENSOR, 1, 7000000}}, 4, 0},
    {"more beside a long one", FP8, F32, ADAM, ECO_MODE_ECO, {{8, TENSOR, 1408, 2048}, {1, TENSOR, 1, 7000000}}, 6, 20},
    {"a long one, SGDM", FP8, F32, SGDM, ECO_MODE_ECO, {{1, TENSOR, 1, 7000000}}, 4, 0},
    {"a longer one, SGDM", FP8, F32, SGDM, ECO_MODE_ECO, {{1, TENSOR, 1, 70000000}}, 4, 5},
};

int main(void) {
  static eco_tensor_t list[1024];
  int bad = 0;
  for (size_t c = 0; c < sizeof cases / sizeof *cases; ++c) {
    const Case *k = &cases[c];
    size_t n = 0;
    memset(list, 0, sizeof list);
    for (int g = 0; g < 3; ++g)
      for (int i = 0; i < k->t[g].count; ++i, ++n) {
        eco_tensor_t *t = &list[n];
        t->weights = (void *)0x1000; t->scales = (void *)0x2000; t->grad = (void *)0x3000; t->m = (void *)0x4000; t->v = (void *)0x5000; t->aux = (void *)0x6000;
        t->numel = k->t[g].rows * k->t[g].cols;
        t->group_size = k->t[g].scale == ROW ? k->t[g].cols : k->t[g].scale == TENSOR ? t->numel : k->t[g].scale == PLAIN ? 0 : (uint64_t)k->t[g].scale;
        t->tensor_id = (uint32_t)n;
        t->fmt = k->t[g].scale == PLAIN ? ECO_FMT_BF16_PLAIN : k->fmt;
      }
    eco_hparams_t hp;
    memset(&hp, 0, sizeof hp);
    hp.opt = k->opt; hp.mode = k->mode; hp.block_size = 128; hp.state_dtype = hp.scale_dtype = k->state;
    hp.lr = 1e-3; hp.beta1 = 0.9; hp.beta2 = 0.999; hp.eps = 1e-8; hp.step = 1;
    eco_plan_t *plan = NULL;
    if (eco_plan_create(list, n, &hp, &plan) != ECO_OK) { printf("FAILED: %s: %s\n", k->what, eco_last_error()); return 1; }
    for (int again = 0; again < 2; ++again) {
      launches = 0;
      if (eco_step(plan, &hp, NULL) != ECO_OK) { printf("FAILED: %s: %s\n", k->what, eco_last_error()); return 1; }
      int capped = 0;
      for (int i = 0; i < launches && i < MOST; ++i) capped |= (lds_of[i] != 0) << i;
      if (launches != k->launches || capped != k->capped) {
        printf("%s: %d launches, capped %d; expected %d, %d\n", k->what, launches, capped, k->launches, k->capped);
        ++bad;
      }
    }
    (void)eco_plan_destroy(plan);
  }
  /* Without a plan: rows of 1408 are a workgroup of three waves each from 96 MB on, and four to one of eleven where the static tables
   * hold no more.  Short tensors of odd length with one scale are along with longer ones. */
  eco_hparams_t hp;
  memset(&hp, 0, sizeof hp);
  hp.opt = ADAM; hp.mode = ECO_MODE_ECO; hp.block_size = 128; hp.lr = 1e-3; hp.beta1 = 0.9; hp.beta2 = 0.999; hp.eps = 1e-8; hp.step = 1;
  for (int wide = 0; wide < 2; ++wide) {
    memset(list, 0, sizeof list);
    list[0].weights = (void *)0x1000; list[0].scales = (void *)0x2000; list[0].grad = (void *)0x3000; list[0].m = (void *)0x4000; list[0].v = (void *)0x5000;
    list[0].numel = (wide ? 1ull << 21 : 1ull << 19) * 1408;
    list[0].group_size = 1408;
    launches = 0;
    if (eco_step_tensors_noalloc(list, 1, &hp, NULL) != ECO_OK) { printf("FAILED: no plan: %s\n", eco_last_error()); return 1; }
    if (launches != 2 || grid_of[1] != 1u << 19 || block_of[1] != (wide ? 704u : 192u)) {
      printf("no plan, rows of 1408: %d launches, %u workgroups of %u threads\n", launches, grid_of[1], block_of[1]);
      ++bad;
    }
  }
  list[1] = list[0];
  list[0].numel = 10240 * 1024; list[0].group_size = 1024;
  list[1].numel = 6871 * 768; list[1].group_size = 768;
  launches = 0;
  if (eco_step_tensors_noalloc(list, 2, &hp, NULL) != ECO_OK || launches != 2 || grid_of[1] != 10240 + 6871 || block_of[1] != 128) {
    printf("no plan, rows of 1024 and of 768: %d launches, %u workgroups of %u threads\n", launches, grid_of[1], block_of[1]);
    ++bad;
  }
  for (int i = 0; i < 12; ++i) {
    list[i] = list[0];
    list[i].numel = list[i].group_size = i < 2 ? 11942 : 770;
    list[i].tensor_id = (uint32_t)i;
  }
  list[12] = list[13] = list[0];
  list[12].numel = 512; list[12].fmt = ECO_FMT_BF16_PLAIN;
  list[13].numel = list[13].group_size = 1152;
  for (int n = 12; n <= 14; ++n) {
    launches = 0;
    const int tensorwise = n == 12 ? 1 : n == 13 ? 2 : 2;             /* behind the tables' launch and that of the norm and the row */
    if (eco_step_tensors_noalloc(list, (size_t)n, &hp, NULL) != ECO_OK || launches != 4 + tensorwise || grid_of[tensorwise] != 2 * 24 + 10 * 2) {
      printf("no plan, short tensors of odd length, %d: %d launches, %u tiles\n", n, launches, grid_of[tensorwise]);
      ++bad;
    }
  }
  /* Arrays past the caches, all beginning on lines of memory: an array off a line, of those that the step uses, takes it the usual way;
   * what stands in the place of an array that it does not use changes nothing. */
  static const struct { int fmt, opt, mode, v, aux; } uses[] = {{FP8, SGDM, ECO_MODE_ECO, 0, 0}, {FP8, ADAM, ECO_MODE_ECO, 1, 0}, {FP8, SGDM, ECO_MODE_EXACT, 0, 1},
      {FP8, ADAM, ECO_MODE_MASTER, 1, 1}, {ECO_FMT_BF16_PLAIN, ADAM, ECO_MODE_MASTER, 1, 0}, {ECO_FMT_BF16_PLAIN, SGDM, ECO_MODE_EXACT, 0, 0}};
  for (size_t c = 0; c < sizeof uses / sizeof *uses; ++c)
    for (int group = 128; group <= 1024; group += 896)
      for (int planned = 0; planned < 2; ++planned) {
        const void *kernels[4];
        for (int off = 0; off < 4; ++off) {                      /* none, grad, v, aux */
          eco_plan_t *plan = NULL;
          memset(list, 0, sizeof *list);
          list[0].weights = (void *)0x1000; list[0].scales = (void *)0x2000; list[0].m = (void *)0x4000;
          list[0].grad = (void *)(uintptr_t)(off == 1 ? 0x3010 : 0x3000);
          list[0].v = (void *)(uintptr_t)(off == 2 ? (uses[c].v ? 0x5010 : 0x5001) : 0x5000);
          list[0].aux = (void *)(uintptr_t)(off == 3 ? (uses[c].aux ? 0x6010 : 0x6001) : 0x6000);
          list[0].numel = 1 << 26; list[0].group_size = (uint64_t)group; list[0].fmt = uses[c].fmt;
          hp.opt = uses[c].opt; hp.mode = uses[c].mode;
          launches = 0;
          if (planned && eco_plan_create(list, 1, &hp, &plan) != ECO_OK) { printf("FAILED: lines: %s\n", eco_last_error()); return 1; }
          if ((planned ? eco_step(plan, &hp, NULL) : eco_step_tensors_noalloc(list, 1, &hp, NULL)) != ECO_OK) { printf("FAILED: lines: %s\n", eco_last_error()); return 1; }
          kernels[off] = kernel_of[launches - 1];
          if (plan) (void)eco_plan_destroy(plan);
        }
        if (kernels[1] == kernels[0] || (kernels[2] == kernels[0]) != !uses[c].v || (kernels[3] == kernels[0]) != !uses[c].aux) {
          printf("lines of memory, case %zu, groups of %d, %s plan: v %d, aux %d\n", c, group, planned ? "with" : "without", kernels[2] == kernels[0], kernels[3] == kernels[0]);
          ++bad;
        }
      }
  /* Where the streamed kernels begin: steps of fp32 state on either side of 310 MB, of bf16 state of 384 MB. */
  for (int bf16 = 0; bf16 < 2; ++bf16)
    for (int group = 128; group <= 1024; group += 896) {
      const void *kernels[3];
      for (int k = 0; k < 3; ++k) {
        eco_plan_t *plan = NULL;
        memset(list, 0, sizeof *list);
        list[0].weights = (void *)0x1000; list[0].scales = (void *)0x2000; list[0].grad = (void *)0x3000; list[0].m = (void *)0x4000; list[0].v = (void *)0x5000;
        list[0].group_size = (uint64_t)group; list[0].fmt = FP8;
        list[0].numel = (uint64_t)((bf16 ? 384e6 / 7 : 310e6 / 11) * (k == 0 ? 0.5 : k == 1 ? 0.97 : 1.01)) / 16384 * 16384;
        hp.opt = ADAM; hp.mode = ECO_MODE_ECO; hp.state_dtype = bf16;
        launches = 0;
        if (eco_plan_create(list, 1, &hp, &plan) != ECO_OK || eco_step(plan, &hp, NULL) != ECO_OK) { printf("FAILED: line: %s\n", eco_last_error()); return 1; }
        kernels[k] = kernel_of[launches - 1];
        (void)eco_plan_destroy(plan);
      }
      hp.state_dtype = 0;
      if (kernels[0] != kernels[1] || kernels[1] == kernels[2]) { printf("where streaming begins, groups of %d, %s state\n", group, bf16 ? "bf16" : "fp32"); ++bad; }
    }
  /* Launch options hold for the next step of a plan made before they were set, and no longer than they are set. */
  hp.opt = ADAM; hp.mode = ECO_MODE_ECO;
  for (int group = 128; group <= 1024; group += 896) {
    eco_plan_t *plan = NULL;
    memset(list, 0, sizeof *list);
    list[0].weights = (void *)0x1000; list[0].scales = (void *)0x2000; list[0].grad = (void *)0x3000; list[0].m = (void *)0x4000; list[0].v = (void *)0x5000;
    list[0].numel = 1 << 27; list[0].group_size = (uint64_t)group;
    if (eco_plan_create(list, 1, &hp, &plan) != ECO_OK) { printf("FAILED: options: %s\n", eco_last_error()); return 1; }
    size_t lds[3] = {0};
    for (int k = 0; k < 3; ++k) {
      if (eco_set_option(1, k == 1 ? 1536 : -1) != ECO_OK || eco_set_option(2, k == 1 ? 768 : -1) != ECO_OK) return 1;
      launches = 0;
      if (eco_step(plan, &hp, NULL) != ECO_OK) { printf("FAILED: options: %s\n", eco_last_error()); return 1; }
      lds[k] = launches == 1 ? lds_of[0] : 0;
    }
    (void)eco_plan_destroy(plan);
    if (lds[1] != 1536 || lds[0] == 1536 || lds[0] == 0 || lds[2] != lds[0]) {
      printf("options, groups of %d: %zu, %zu, %zu bytes of LDS\n", group, lds[0], lds[1], lds[2]);
      ++bad;
    }
  }
  if (bad) return 1;
  printf("routes ok\n");
  return 0;
}
