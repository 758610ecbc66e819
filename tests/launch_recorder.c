/* Stands in for the HIP calls that launch kernels, in a process without a GPU: notes which kernel the library would have
 * launched and launches nothing.  Loaded before the library, with its symbols visible to it. */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <stddef.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3_t;
enum { MAX_LAUNCHES = 256 };
static char names[MAX_LAUNCHES][512];
static unsigned grids[MAX_LAUNCHES][2];
static int count, lds_limit_fails;

int hipLaunchKernel(const void *f, dim3_t grid, dim3_t block, void **args, size_t lds, void *stream) {
  Dl_info info;
  (void)block; (void)args; (void)lds; (void)stream;
  if (count < MAX_LAUNCHES) {
    names[count][0] = 0;
    if (dladdr(f, &info) && info.dli_sname) strncpy(names[count], info.dli_sname, sizeof names[0] - 1);
    grids[count][0] = grid.x;
    grids[count][1] = grid.y;
    ++count;
  }
  return 0;
}
/* the halves of a <<<>>> launch around the stub that calls hipLaunchKernel */
static dim3_t pushed_grid, pushed_block;
static size_t pushed_lds;
static void *pushed_stream;
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void *stream) {
  pushed_grid = grid; pushed_block = block; pushed_lds = lds; pushed_stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3_t *grid, dim3_t *block, size_t *lds, void **stream) {
  *grid = pushed_grid; *block = pushed_block; *lds = pushed_lds; *stream = pushed_stream;
  return 0;
}
int hipFuncSetAttribute(const void *f, int attr, int value) {
  (void)f; (void)attr; (void)value;
  return lds_limit_fails ? 1 : 0;
}
int hipGetDevice(int *dev) { *dev = 0; return 0; }
int hipGetLastError(void) { return 0; }

void recorder_reset(int fail) { count = 0; lds_limit_fails = fail; }
int recorder_count(void) { return count; }
const char *recorder_name(int i) { return names[i]; }
unsigned recorder_grid(int i, int k) { return grids[i][k]; }
