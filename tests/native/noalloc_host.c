/* eco_step_tensors_noalloc allocates nothing on the host either: this program's operator new stands before the C++
 * library's and counts.  No GPU is needed: launches and the two queries that the call makes end here. */
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <hip/hip_runtime_api.h>

#include "eco.h"

static int allocations = 0, launches = 0;

void *_Znwm(size_t n) { ++allocations; return malloc(n); }
void *_Znam(size_t n) { ++allocations; return malloc(n); }

hipError_t hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds, hipStream_t stream) {
  (void)f; (void)grid; (void)block; (void)args; (void)lds; (void)stream;
  ++launches;
  return hipSuccess;
}
/* what a launch statement calls around it */
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream) {
  (void)grid; (void)block; (void)lds; (void)stream;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *stream) {
  grid->x = grid->y = grid->z = block->x = block->y = block->z = 1;
  *lds = 0;
  *stream = NULL;
  return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGetDevice(int *device) { *device = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *x, hipDeviceAttribute_t a, int device) { (void)a; (void)device; *x = 256; return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *symbol) { (void)symbol; *p = (void *)0x100000; return hipSuccess; }

int main(void) {
  static const uint64_t lengths[3] = {5000, 333 * 777, 1408};
  eco_tensor_t list[200];
  memset(list, 0, sizeof list);
  for (int i = 0; i < 200; ++i) {
    eco_tensor_t *t = &list[i];
    t->weights = (void *)0x1000; t->scales = (void *)0x2000; t->grad = (void *)0x3000; t->m = (void *)0x4000; t->v = (void *)0x5000;
    t->numel = lengths[i % 3];
    t->group_size = i % 3 == 2 ? 1408 : 0;
    t->tensor_id = (uint32_t)i;
    t->fmt = i % 7 == 6 ? ECO_FMT_BF16_PLAIN : i % 2 ? ECO_FMT_INT4 : ECO_FMT_FP8_E4M3;
  }
  eco_hparams_t hp;
  memset(&hp, 0, sizeof hp);
  hp.opt = ECO_OPT_ADAM; hp.mode = ECO_MODE_ECO; hp.block_size = 128;
  hp.lr = 1e-3; hp.beta1 = 0.9; hp.beta2 = 0.999; hp.eps = 1e-8; hp.step = 1;
  /* a short list (arguments of one kernel for each format), one of the most tensors of that kind, lists with tables */
  for (int n = 1; n <= 200; n += n < 100 ? 1 : 50) {
    allocations = launches = 0;
    const eco_status_t st = eco_step_tensors_noalloc(list, (size_t)n, &hp, NULL);
    if (st != ECO_OK || launches == 0) { printf("FAILED: %d tensors: status %d, %d launches (%s)\n", n, st, launches, eco_last_error()); return 1; }
    if (allocations) { printf("FAILED: %d tensors: %d allocations\n", n, allocations); return 1; }
  }
  printf("no host allocation\n");
  return 0;
}
