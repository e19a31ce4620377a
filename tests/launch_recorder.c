/* Stands in for HIP's launch calls and prints every launch: threads per block, blocks, and the
 * kernel's first RECORDED_ARGS arguments as 64-bit words. Nothing runs. */
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct {
  uint32_t x, y, z;
} dim3;

static dim3 grid, block;
static size_t shared;
static void *stream;

int __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, void *s) {
  grid = g;
  block = b;
  shared = lds;
  stream = s;
  return 0;
}

int __hipPopCallConfiguration(dim3 *g, dim3 *b, size_t *lds, void **s) {
  *g = grid;
  *b = block;
  *lds = shared;
  *s = stream;
  return 0;
}

int hipLaunchKernel(const void *f, dim3 g, dim3 b, void **args, size_t lds, void *s) {
  (void)f;
  (void)lds;
  (void)s;
  printf("%u %u", b.x * b.y * b.z, g.x);
  const int n = atoi(getenv("RECORDED_ARGS"));
  for (int i = 0; i < n; ++i) {
    uint64_t word = 0;
    memcpy(&word, args[i], 8);
    printf(" %llu", (unsigned long long)word);
  }
  printf("\n");
  fflush(stdout);
  return 0;
}

int hipGetLastError(void) { return 0; }
