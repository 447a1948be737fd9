/* A HIP runtime without a device, for the host code of the verifier's library: it hands out host memory, launches nothing, keeps a list
 * of what was asked for, and lets one call fail.  Loaded with global visibility before the library, whose calls then come here. */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;
enum { kFunctions = 256, kLog = 1 << 16 };
static const void* functions[kFunctions];
static const char* names[kFunctions];
static int function_count;
static size_t allowed[kFunctions];                     /* dynamic LDS, as hipFuncSetAttribute set it */
static int over;                                       /* launches with more than 64 KB and more than was set */
static char log_[kLog];
static size_t log_used;
static char fail_name[64];
static int fail_in;
static int last_error;                                 /* kept until hipGetLastError */

/* The fail_after-th next call of `name` (0: the next one) returns an error. */
void recorded_fail(const char* name, int fail_after) { snprintf(fail_name, sizeof fail_name, "%s", name); fail_in = fail_after + 1; }
const char* recorded_log(void) { return log_; }
void recorded_clear(void) { log_used = 0; log_[0] = 0; fail_name[0] = 0; }

static int note(const char* name, const char* what) {
    const int n = snprintf(log_ + log_used, kLog - log_used, "%s %s\n", name, what);
    if (n > 0 && log_used + (size_t)n < kLog) log_used += (size_t)n;
    if (strcmp(name, fail_name) == 0 && --fail_in == 0) { fail_name[0] = 0; return last_error = 999; }
    return 0;
}

void** __hipRegisterFatBinary(const void* data) { static void* module; (void)data; return &module; }
void __hipUnregisterFatBinary(void** modules) { (void)modules; }
void __hipRegisterFunction(void** modules, const void* host, char* device, const char* name, unsigned limit, void* tid, void* bid, dim3* block,
                           dim3* grid, int* w) {
    (void)modules; (void)device; (void)limit; (void)tid; (void)bid; (void)block; (void)grid; (void)w;
    if (function_count < kFunctions) { functions[function_count] = host; names[function_count++] = name; }
}
void __hipRegisterVar(void** modules, void* var, char* host, char* device, int ext, size_t size, int constant, int global) {
    (void)modules; (void)var; (void)host; (void)device; (void)ext; (void)size; (void)constant; (void)global;
}
static struct { dim3 grid, block; size_t lds; void* stream; } pushed;
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void* stream) {
    pushed.grid = grid; pushed.block = block; pushed.lds = lds; pushed.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, void** stream) {
    *grid = pushed.grid; *block = pushed.block; *lds = pushed.lds; *stream = pushed.stream;
    return 0;
}
int hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t lds, void* stream) {
    (void)block; (void)args; (void)stream;
    for (int i = 0; i < function_count; ++i)
        if (functions[i] == f) {
            char what[256];
            over += lds > 65536 && lds > allowed[i];
            snprintf(what, sizeof what, "%.200s %u", names[i], grid.x);
            return note("launch", what);
        }
    return note("launch", "?");
}
int hipGetLastError(void) { const int e = last_error; last_error = 0; return e; }
int hipGetDevice(int* device) { *device = 0; return 0; }
int recorded_over(void) { return over; }
int hipFuncSetAttribute(const void* f, int attribute, int value) {
    (void)attribute;
    for (int i = 0; i < function_count; ++i) if (functions[i] == f) allowed[i] = (size_t)value;
    return 0;
}
int hipGetSymbolAddress(void** p, const void* symbol) { (void)symbol; *p = log_; return 0; }
int hipMalloc(void** p, size_t size) { *p = calloc(1, size); return *p ? note("malloc", "") : 2; }
int hipFree(void* p) { free(p); return 0; }
int hipHostMalloc(void** p, size_t size, unsigned flags) { (void)flags; *p = calloc(1, size); return *p ? note("host_malloc", "") : 2; }
int hipHostFree(void* p) { free(p); return 0; }
int hipMemcpyAsync(void* to, const void* from, size_t size, int kind, void* stream) {
    (void)stream;
    const int rc = note(kind == 1 ? "to_device" : (kind == 2 ? "to_host" : "copy"), "");
    if (rc == 0) memcpy(to, from, size);
    return rc;
}
int hipStreamSynchronize(void* stream) { (void)stream; return note("synchronize", ""); }
int hipEventCreate(void** e) { static int event; *e = &event; return 0; }
int hipEventDestroy(void* e) { (void)e; return 0; }
int hipEventRecord(void* e, void* stream) { (void)e; (void)stream; return 0; }
int hipEventSynchronize(void* e) { (void)e; return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 0.f; return 0; }
