/* Stands in front of the HIP runtime (LD_PRELOAD) and writes down the calls that the library's host code makes.  Nothing
 * reaches a device: launches and attributes succeed and do nothing, the device is number 0 with 256 compute units. */
#include <stddef.h>
#include <stdint.h>

struct call {
  int32_t kind;             /* one of the below */
  int32_t grid;             /* launch: workgroups */
  const void *kernel;       /* attribute, launch */
  int64_t bytes;            /* attribute: the limit; launch: dynamic LDS */
  const void *stream;       /* launch */
};
enum { SET_ATTRIBUTE = 1, LAUNCH, GET_DEVICE, DEVICE_ATTRIBUTE, SYMBOL_ADDRESS };
struct dim3_ {
  uint32_t x, y, z;
};

enum { ROOM = 4096 };
static struct call calls[ROOM];
static int n_calls;
static char symbols[1 << 16];

static void write_down(struct call c) {
  if (n_calls < ROOM) calls[n_calls++] = c;
}

__attribute__((visibility("default"))) int recorded(struct call *to) {
  const int n = n_calls;
  for (int i = 0; i < n; ++i) to[i] = calls[i];
  n_calls = 0;
  return n;
}

__attribute__((visibility("default"))) int hipFuncSetAttribute(const void *f, int attribute, int value) {
  (void)attribute;
  write_down((struct call){SET_ATTRIBUTE, 0, f, value, NULL});
  return 0;
}
__attribute__((visibility("default"))) int hipLaunchKernel(const void *f, struct dim3_ grid, struct dim3_ block, void **args,
                                                           size_t lds, void *stream) {
  (void)block;
  (void)args;
  write_down((struct call){LAUNCH, (int32_t)grid.x, f, (int64_t)lds, stream});
  return 0;
}
__attribute__((visibility("default"))) int hipGetDevice(int *device) {
  write_down((struct call){GET_DEVICE, 0, NULL, 0, NULL});
  *device = 0;
  return 0;
}
__attribute__((visibility("default"))) int hipDeviceGetAttribute(int *value, int attribute, int device) {
  (void)attribute;
  (void)device;
  write_down((struct call){DEVICE_ATTRIBUTE, 0, NULL, 0, NULL});
  *value = 256;
  return 0;
}
__attribute__((visibility("default"))) int hipGetSymbolAddress(void **address, const void *symbol) {
  (void)symbol;
  write_down((struct call){SYMBOL_ADDRESS, 0, NULL, 0, NULL});
  *address = symbols;
  return 0;
}
