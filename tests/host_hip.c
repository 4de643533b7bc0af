/* The HIP runtime calls of libgg.so on host memory: allocations and copies
 * work, kernels are accepted and never run, and a stream or event that is asked
 * answers what the test set.  Loaded before libgg.so with global symbols. */
#include <stdlib.h>
#include <string.h>

static int answer = 600;       /* hipErrorNotReady */
static size_t limit = 1 << 30; /* bytes that one allocation may have */
static long launches = 0;

void host_hip_answer(int e) { answer = e; }
void host_hip_limit(size_t bytes) { limit = bytes; }
long host_hip_launches(void) { return launches; }

void* __hipRegisterFatBinary(const void* p) { return (void*)p; }
void __hipUnregisterFatBinary(void* p) { (void)p; }
void __hipRegisterFunction() {}
void __hipRegisterVar() {}
int __hipPushCallConfiguration() { return 0; }
int __hipPopCallConfiguration() { return 0; }
int hipLaunchKernel() { return launches++, 0; }

int hipMalloc(void** p, size_t n) { return n > limit ? 2 : (*p = calloc(1, n)) ? 0 : 2; }
int hipHostMalloc(void** p, size_t n, unsigned f) { return (void)f, hipMalloc(p, n); }
int hipFree(void* p) { return free(p), 0; }
int hipHostFree(void* p) { return free(p), 0; }
int hipMemcpy(void* d, const void* s, size_t n, int k) { return (void)k, memcpy(d, s, n), 0; }
int hipMemcpyAsync(void* d, const void* s, size_t n, int k, void* st) { return (void)st, hipMemcpy(d, s, n, k); }
int hipMemcpyWithStream(void* d, const void* s, size_t n, int k, void* st) { return (void)st, hipMemcpy(d, s, n, k); }
int hipMemset(void* d, int v, size_t n) { return memset(d, v, n), 0; }
int hipMemsetAsync(void* d, int v, size_t n, void* st) { return (void)st, hipMemset(d, v, n); }

int hipStreamQuery(void* s) { return (void)s, answer; }
int hipEventQuery(void* e) { return (void)e, answer; }
int hipStreamSynchronize(void* s) { return (void)s, answer == 600 ? 0 : answer; }
int hipEventSynchronize(void* e) { return (void)e, answer == 600 ? 0 : answer; }
int hipDeviceSynchronize(void) { return answer == 600 ? 0 : answer; }

static int any;
int hipEventCreate(void** e) { return *e = &any, 0; }
int hipEventCreateWithFlags(void** e, unsigned f) { return (void)f, hipEventCreate(e); }
int hipStreamCreateWithFlags(void** s, unsigned f) { return (void)f, hipEventCreate(s); }
int hipEventRecord() { return 0; }
int hipEventDestroy() { return 0; }
int hipStreamDestroy() { return 0; }
int hipStreamWaitEvent() { return 0; }
int hipFuncSetAttribute() { return 0; }
int hipSetDevice() { return 0; }
int hipGetLastError(void) { return 0; }
int hipGetDevice(int* d) { return *d = 0; }
int hipGetDevicePropertiesR0600() { return 1; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n) { return *n = 1, 0; }
