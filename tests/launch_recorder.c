/* The HIP runtime's calls that a launch makes, recorded instead of run: loaded
 * before libhcmix.so in a process of its own, so that a test sees the grid of
 * every launch of a call (and the first bytes of its first argument) without a
 * GPU and without memory behind the operands. */
#include <stddef.h>
#include <stdint.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3_t;
typedef struct { dim3_t grid, block; uint64_t arg[2]; } launch_t;

enum { MOST = 64 };
launch_t launches[MOST];
int launch_count;

static struct { dim3_t grid, block; size_t lds; void *stream; } config;

int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void *stream) {
  config.grid = grid;
  config.block = block;
  config.lds = lds;
  config.stream = stream;
  return 0;
}

int __hipPopCallConfiguration(dim3_t *grid, dim3_t *block, size_t *lds, void **stream) {
  *grid = config.grid;
  *block = config.block;
  *lds = config.lds;
  *stream = config.stream;
  return 0;
}

int hipLaunchKernel(const void *kernel, dim3_t grid, dim3_t block, void **args, size_t lds,
                    void *stream) {
  (void)kernel, (void)lds, (void)stream;
  if (launch_count < MOST) {
    launch_t *l = &launches[launch_count];
    l->grid = grid;
    l->block = block;
    memcpy(&l->arg[0], args[0], 8);   /* every kernel's first argument starts with a pointer */
  }
  launch_count++;
  return 0;
}

int hipGetLastError(void) { return 0; }
int hipGetDevice(int *device) { *device = 0; return 0; }
int hipFuncSetAttribute(const void *kernel, int attribute, int value) {
  (void)kernel, (void)attribute, (void)value;
  return 0;
}
