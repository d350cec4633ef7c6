/* Stands in for the HIP runtime in a process without a GPU: kernel launches of the library are written to a list (name,
 * grid, block, two leading integer arguments behind the first) instead of being enqueued.  Loaded with RTLD_GLOBAL in front of the
 * library, so that the library's calls bind to the definitions here (see launches.py). */
#include <stdint.h>
#include <stdio.h>
#include <string.h>

typedef struct { unsigned x, y, z; } dim3_t;
typedef struct { char name[512]; dim3_t grid, block; int32_t arg1, arg2; } record_t;

static record_t records[256];
static int n_records;
static struct { const void *stub; char name[512]; } kernels[1024];
static int n_kernels;
static dim3_t cfg_grid, cfg_block;
static size_t cfg_shmem;
static void *cfg_stream;
static void (*event_hook)(void);
static int last_error, failing;

int rec_count(void) { return n_records; }
const record_t *rec_get(int i) { return &records[i]; }
void rec_reset(void) { n_records = 0; }
void rec_set_error(int pending, int of_launches) { last_error = pending; failing = of_launches; }   /* left by the program before; what every launch fails with */
int rec_error(void) { return last_error; }
void rec_on_event(void (*hook)(void)) { event_hook = hook; }   /* called by every hipEventRecord */

/* what the code of a HIP object calls when it is loaded */
static void *module_handle;
void **__hipRegisterFatBinary(const void *data) { (void)data; return &module_handle; }
void __hipUnregisterFatBinary(void **modules) { (void)modules; }
void __hipRegisterFunction(void **modules, const void *stub, char *device_function, const char *device_name, unsigned threads, void *tid,
                           void *bid, void *block, void *grid, int *wave)
{
    (void)modules; (void)device_function; (void)threads; (void)tid; (void)bid; (void)block; (void)grid; (void)wave;
    if (n_kernels < 1024) {
        kernels[n_kernels].stub = stub;
        snprintf(kernels[n_kernels].name, sizeof kernels[n_kernels].name, "%s", device_name);
        ++n_kernels;
    }
}
void __hipRegisterVar(void **modules, void *var, char *host, char *device, int ext, size_t size, int constant, int global)
{
    (void)modules; (void)var; (void)host; (void)device; (void)ext; (void)size; (void)constant; (void)global;
}

/* a launch */
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t shmem, void *stream)
{
    cfg_grid = grid; cfg_block = block; cfg_shmem = shmem; cfg_stream = stream;
    return 0;
}
int __hipPopCallConfiguration(dim3_t *grid, dim3_t *block, size_t *shmem, void **stream)
{
    *grid = cfg_grid; *block = cfg_block; *shmem = cfg_shmem; *stream = cfg_stream;
    return 0;
}
int hipLaunchKernel(const void *stub, dim3_t grid, dim3_t block, void **args, size_t shmem, void *stream)
{
    (void)shmem; (void)stream;
    if (failing) return last_error = failing;
    if (n_records >= 256) return 1;
    record_t *r = &records[n_records++];
    r->name[0] = 0; r->arg1 = r->arg2 = -1;
    for (int i = 0; i < n_kernels; ++i)
        if (kernels[i].stub == stub) memcpy(r->name, kernels[i].name, sizeof r->name);
    r->grid = grid; r->block = block;
    if (strstr(r->name, "paged_attention_blocks_kernel")) {   /* (AttnArgs, int, int) */
        memcpy(&r->arg1, args[1], 4);
        memcpy(&r->arg2, args[2], 4);
    }
    return 0;
}
int hipGetLastError(void) { const int e = last_error; last_error = 0; return e; }
int hipGetDevice(int *dev) { *dev = 0; return 0; }
int hipEventCreate(void **e) { static int token; *e = &token; return 0; }
int hipEventDestroy(void *e) { (void)e; return 0; }
int hipEventSynchronize(void *e) { (void)e; return 0; }
int hipEventElapsedTime(float *ms, void *a, void *b) { (void)a; (void)b; *ms = 0.f; return 0; }
int hipEventRecord(void *e, void *stream)
{
    (void)e; (void)stream;
    if (event_hook) event_hook();
    return 0;
}
