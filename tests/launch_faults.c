/* Stands in for the HIP calls of a sweep on a machine without a device: launches
 * are counted and do nothing, and one of them fails. */
#include <stddef.h>
#include <stdint.h>

typedef struct { uint32_t x, y, z; } dim3_t;
static long count, fail_at;
static int last;

void faults_reset(long n) { count = 0; fail_at = n; last = 0; }
long faults_count(void) { return count; }

int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void* stream) {
  (void)grid; (void)block; (void)lds; (void)stream;
  return 0;
}
int __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* lds, void** stream) {
  const dim3_t one = {1, 1, 1};
  *grid = *block = one;
  *lds = 0;
  *stream = NULL;
  return 0;
}
int hipLaunchKernel(const void* f, dim3_t grid, dim3_t block, void** args, size_t lds, void* stream) {
  (void)f; (void)grid; (void)block; (void)args; (void)lds; (void)stream;
  last = ++count == fail_at ? 719 : 0; /* hipErrorLaunchFailure */
  return last;
}
int hipGetLastError(void) { const int e = last; last = 0; return e; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipFuncSetAttribute(const void* f, int attr, int value) { (void)f; (void)attr; (void)value; return 0; }
