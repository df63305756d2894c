/* Stands in for the HIP runtime where a test wants to see what the library would launch, without a GPU: loaded in front of
 * the real runtime, it keeps every launch and answers the few other calls that the library makes. */
#include <stddef.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3;
typedef struct { const char* name; dim3 grid, block; size_t lds; unsigned words[32]; } launch;   /* words: the first argument's first 128 bytes */

static struct { const void* host; const char* name; } kernels[512];
static int n_kernels, n_launches, device_error, attribute_error;
static launch launches[256];
static struct { dim3 grid, block; size_t lds; void* stream; } next;
static char symbol[256];

void** __hipRegisterFatBinary(const void* data) { static void* module; (void)data; return &module; }
void __hipUnregisterFatBinary(void** module) { (void)module; }
void __hipRegisterVar() {}
void __hipRegisterFunction(void** module, const void* host, char* device, const char* name)
{
    (void)module; (void)device;
    if (n_kernels < 512) { kernels[n_kernels].host = host; kernels[n_kernels++].name = name; }
}
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void* stream)
{
    next.grid = grid; next.block = block; next.lds = lds; next.stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, void** stream)
{
    *grid = next.grid; *block = next.block; *lds = next.lds; *stream = next.stream;
    return 0;
}
int hipLaunchKernel(const void* host, dim3 grid, dim3 block, void** args, size_t lds, void* stream)
{
    (void)stream;
    launch l = {"?", grid, block, lds};
    memcpy(l.words, args[0], sizeof(l.words));          /* (past a shorter argument lies the caller's own stack) */
    for (int i = 0; i < n_kernels; ++i) if (kernels[i].host == host) l.name = kernels[i].name;
    if (n_launches < 256) launches[n_launches++] = l;
    return 0;
}
int hipFuncSetAttribute(const void* host, int attribute, int value) { (void)host; (void)attribute; (void)value; return attribute_error; }
int hipGetDevice(int* device) { *device = 0; return device_error; }
int hipGetLastError(void) { return 0; }
int hipGetSymbolAddress(void** at, const void* what) { (void)what; *at = symbol; return 0; }

void recorder_errors(int device, int attribute) { device_error = device; attribute_error = attribute; }
int recorder_take(launch* out)
{
    const int n = n_launches;
    memcpy(out, launches, sizeof(launch) * n);
    n_launches = 0;
    return n;
}
