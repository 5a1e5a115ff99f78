/* A stand-in for the HIP runtime that libgka links against, preloaded into a process without a GPU: it launches nothing
 * and writes down what the library asked for. One line per call on the file of recorder_open():
 *   launch <kernel's mangled name> <grid> <block> <dynamic LDS bytes>
 *   attribute <kernel's mangled name> <attribute> <value> <device>
 *   variable <device variable's name> <bytes> 0 0     (when its address, RECORDER_VARIABLE, is asked for)
 * and after recorder_words(n), behind each launch, the first n 8-byte words of its first argument (the kernels take one struct,
 * which the launch has copied to the stack; what follows a shorter one are the callers' variables):
 *   words <value> ...
 */
#include <stdio.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>

#define RECORDER_VARIABLE ((uintptr_t)1 << 60)

typedef struct { uint32_t x, y, z; } dim3_t;

static struct { const void *host; const char *name; } kernels[4096];
static int n_kernels, device, n_words;
static struct { const void *host; const char *name; size_t size; } variables[64];
static int n_variables;
static FILE *out;
static struct { dim3_t grid, block; size_t lds; void *stream; } pushed;

void recorder_open(const char *path) { out = fopen(path, "w"); }
void recorder_close(void) { if (out) fclose(out); out = NULL; }
void recorder_set_device(int d) { device = d; }
void recorder_words(int n) { n_words = n; }

static const char *name_of(const void *host)
{
    for (int i = 0; i < n_kernels; ++i)
        if (kernels[i].host == host) return kernels[i].name;
    return "?";
}

void **__hipRegisterFatBinary(const void *data) { (void)data; static void *handle; return &handle; }
void __hipUnregisterFatBinary(void **modules) { (void)modules; }
void __hipRegisterFunction(void **modules, const void *host, char *device_function, const char *device_name,
                           unsigned thread_limit, void *tid, void *bid, void *block, void *grid, int *wsize)
{
    (void)modules; (void)device_function; (void)thread_limit; (void)tid; (void)bid; (void)block; (void)grid; (void)wsize;
    if (n_kernels < 4096) { kernels[n_kernels].host = host; kernels[n_kernels++].name = device_name; }
}
void __hipRegisterVar(void **modules, void *var, char *host, char *dev, int ext, size_t size, int constant, int global)
{
    (void)modules; (void)host; (void)ext; (void)constant; (void)global;
    if (n_variables < 64) { variables[n_variables].host = var; variables[n_variables].name = dev; variables[n_variables++].size = size; }
}
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void *stream)
{
    pushed.grid = grid; pushed.block = block; pushed.lds = lds; pushed.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3_t *grid, dim3_t *block, size_t *lds, void **stream)
{
    *grid = pushed.grid; *block = pushed.block; *lds = pushed.lds; *stream = pushed.stream;
    return 0;
}
int hipLaunchKernel(const void *host, dim3_t grid, dim3_t block, void **args, size_t lds, void *stream)
{
    (void)stream;
    if (out) fprintf(out, "launch %s %u %u %zu\n", name_of(host), grid.x, block.x, lds);
    if (out && n_words > 0) {
        uint64_t word;
        fprintf(out, "words");
        for (int i = 0; i < n_words; ++i) {
            memcpy(&word, (const char *)args[0] + 8 * i, 8);
            fprintf(out, " %llu", (unsigned long long)word);
        }
        fprintf(out, "\n");
    }
    return 0;
}
int hipFuncSetAttribute(const void *host, int attribute, int value)
{
    if (out) fprintf(out, "attribute %s %d %d %d\n", name_of(host), attribute, value, device);
    return 0;
}
int hipGetDevice(int *d) { *d = device; return 0; }
int hipGetLastError(void) { return 0; }
int hipGetSymbolAddress(void **p, const void *symbol)
{
    for (int i = 0; i < n_variables; ++i)
        if (variables[i].host == symbol && out) fprintf(out, "variable %s %zu 0 0\n", variables[i].name, variables[i].size);
    *p = (void *)RECORDER_VARIABLE;
    return 0;
}
int hipEventCreate(void **e) { *e = (void *)1; return 0; }
int hipEventDestroy(void *e) { (void)e; return 0; }
int hipEventRecord(void *e, void *s) { (void)e; (void)s; return 0; }
int hipEventSynchronize(void *e) { (void)e; return 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) { (void)a; (void)b; *ms = 0; return 0; }
