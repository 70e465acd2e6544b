/* A step that stops between its launches, and the next step of the same plan.  The launch that fails is chosen here: this
 * program's hipLaunchKernel stands before the runtime's, passes every launch on but one, and reports that one as failed.
 * After it the tensors are restored and stepped again, with smaller gradients than the stopped step had; the result has to
 * be that of a plan that has never failed, byte for byte.  Tensors with one scale: their maxima live in the plan's scratch. */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <hip/hip_runtime_api.h>

#include "eco.h"

static int countdown = 0, launches = 0;      /* the launch that fails (1 = the next one), launches since it was set */
static hipError_t pending = hipSuccess;

hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t stream) {
  static hipError_t (*next)(const void *, dim3, dim3, void **, size_t, hipStream_t);
  if (!next) *(void **)&next = dlsym(RTLD_NEXT, "hipLaunchKernel");
  ++launches;
  if (countdown && --countdown == 0) return pending = hipErrorUnknown;
  return next(f, grid, block, args, lds, stream);
}

hipError_t hipGetLastError(void) {
  static hipError_t (*next)(void);
  const hipError_t e = pending;
  if (!next) *(void **)&next = dlsym(RTLD_NEXT, "hipGetLastError");
  pending = hipSuccess;
  return e != hipSuccess ? e : next();
}

#define CHECK(c)                                                                                       \
  do {                                                                                                 \
    if (!(c)) { printf("FAILED line %d: %s (%s)\n", __LINE__, #c, eco_last_error()); exit(1); }        \
  } while (0)

/* One pass (with a tail), one pass, two passes, one pass; the others are there because a few small tensors alone, or beside a
 * long one, would not be stepped in one pass: they are set up once and not compared. */
enum { TENSORS = 4, FILL = 7, ARRAYS = 5 };  /* arrays: codes, scale, gradient, m, v */
static const uint64_t numel[TENSORS + FILL] = {20001, 40000, 5000000, 300007, 4700000, 4700000, 4700000, 4700000, 4700000, 4700000, 4700000};
static const size_t width[ARRAYS] = {1, 0, 2, 4, 4};

static size_t bytes_of(int t, int a) { return a == 1 ? 16 : (size_t)numel[t] * width[a] + 16; }

static void *dev[TENSORS + FILL][ARRAYS];
static unsigned char *host[TENSORS][ARRAYS];

static void restore(int gradient_exponent) {
  for (int t = 0; t < TENSORS; ++t)
    for (int a = 0; a < ARRAYS; ++a) {
      unsigned char *h = host[t][a];
      const size_t n = bytes_of(t, a);
      uint32_t x = 12345u + 77u * (uint32_t)t + (uint32_t)a;
      if (a == 1) {
        const float s = 1e-3f;
        memset(h, 0, n);
        memcpy(h, &s, 4);
      } else {
        for (uint64_t i = 0; i < numel[t]; ++i) {
          x = x * 1664525u + 1013904223u;
          if (a == 0) h[i] = (unsigned char)((x >> 24) % 127);                                   /* E4M3, never NaN */
          else if (a == 2) ((uint16_t *)h)[i] = (uint16_t)((x >> 16 & 0x807Fu) | (uint32_t)(127 + gradient_exponent) << 7);
          else ((float *)h)[i] = a == 3 ? ((int)(x >> 8) - (1 << 23)) * 1e-12f : (float)(x >> 8) * 1e-14f + 1e-9f;
        }
      }
      CHECK(hipMemcpy(dev[t][a], h, n, hipMemcpyHostToDevice) == hipSuccess);
    }
}

static unsigned char *result(int t, int a) {
  unsigned char *r = malloc(bytes_of(t, a));
  CHECK(hipMemcpy(r, dev[t][a], bytes_of(t, a), hipMemcpyDeviceToHost) == hipSuccess);
  return r;
}

int main(void) {
  eco_tensor_t list[TENSORS + FILL];
  memset(list, 0, sizeof list);
  for (int t = 0; t < TENSORS + FILL; ++t) {
    for (int a = 0; a < ARRAYS; ++a) {
      CHECK(hipMalloc(&dev[t][a], bytes_of(t, a)) == hipSuccess);
      if (t < TENSORS) CHECK((host[t][a] = calloc(1, bytes_of(t, a))) != NULL);
      else CHECK(hipMemset(dev[t][a], a == 0 ? 0x30 : 0, bytes_of(t, a)) == hipSuccess);
    }
    list[t].weights = dev[t][0]; list[t].scales = dev[t][1]; list[t].grad = dev[t][2]; list[t].m = dev[t][3]; list[t].v = dev[t][4];
    list[t].numel = list[t].group_size = numel[t];
    list[t].tensor_id = (uint32_t)t;
    list[t].fmt = ECO_FMT_FP8_E4M3;
  }
  eco_hparams_t hp;
  memset(&hp, 0, sizeof hp);
  hp.opt = ECO_OPT_SGDM; hp.round = ECO_ROUND_SR; hp.mode = ECO_MODE_ECO; hp.block_size = 128; hp.state_dtype = hp.scale_dtype = ECO_DT_FP32;
  hp.lr = 0.05; hp.beta1 = 0.9; hp.beta2 = 0.999; hp.eps = 1e-8; hp.step = 3; hp.seed = 1;

  eco_plan_t *plan = NULL;
  CHECK(eco_plan_create(list, TENSORS + FILL, &hp, &plan) == ECO_OK);
  restore(-10);
  launches = 0;
  CHECK(eco_step(plan, &hp, NULL) == ECO_OK && hipDeviceSynchronize() == hipSuccess);
  const int all = launches;
  unsigned char *want[TENSORS][ARRAYS];
  for (int t = 0; t < TENSORS; ++t)
    for (int a = 0; a < ARRAYS; ++a) want[t][a] = result(t, a);
  CHECK(eco_plan_destroy(plan) == ECO_OK);
  CHECK(all == 7);                                       /* three for the one-pass tensors, four for the long one */

  int bad = 0;
  for (int stop = 1; stop <= all; ++stop) {
    CHECK(eco_plan_create(list, TENSORS + FILL, &hp, &plan) == ECO_OK);
    restore(2);                                          /* maxima far above those of the step that follows */
    countdown = stop;
    CHECK(eco_step(plan, &hp, NULL) == ECO_EHIP && countdown == 0 && hipDeviceSynchronize() == hipSuccess);
    for (int again = 0; again < 2; ++again) {            /* and the step after that one is an ordinary one */
      restore(-10);
      launches = 0;
      CHECK(eco_step(plan, &hp, NULL) == ECO_OK && hipDeviceSynchronize() == hipSuccess);
      if (again && launches != all) { printf("launch %d stopped: %d launches instead of %d two steps later\n", stop, launches, all); ++bad; }
      for (int t = 0; t < TENSORS; ++t)
        for (int a = 0; a < ARRAYS; ++a) {
          unsigned char *got = result(t, a);
          if (memcmp(got, want[t][a], bytes_of(t, a)) != 0) { printf("launch %d stopped: tensor %d array %d differs\n", stop, t, a); ++bad; }
          free(got);
        }
    }
    CHECK(eco_plan_destroy(plan) == ECO_OK);
    printf("stopped at launch %d of %d\n", stop, all);
    fflush(stdout);
  }
  if (bad) return 1;
  printf("stopped step ok\n");
  return 0;
}
