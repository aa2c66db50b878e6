/* The HIP runtime calls that librinr.so makes, as host stand-ins: allocations come from the heap (those above a limit fail),
 * kernel launches are only written down.  For tests of the library's host side without a GPU; loaded before librinr.so. */
#include <stddef.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;
enum { OK = 0, OUT_OF_MEMORY = 2, N_LAUNCHES = 1024 };

static int last_error;
static size_t malloc_limit = SIZE_MAX;
static int cus = 256, resident = 1;
static size_t cu_lds;                   /* not 0: a CU's LDS, which bounds the workgroups side by side as well */
static int device;                      /* the current GPU */
static char *done;                      /* what touches a GPU's work, with the GPU that was current: "sync 0, copy 0, " */
static size_t done_room;
static int64_t live;                    /* allocations not freed */
static int n_launches;
static uint32_t launches[N_LAUNCHES][4];       /* grid x, y; threads; dynamic LDS */

void fake_set(size_t limit, int n_cus, int n_resident) { malloc_limit = limit; cus = n_cus; resident = n_resident; n_launches = 0; }
void fake_cu_lds(size_t bytes) { cu_lds = bytes; }
int fake_launches(uint32_t *out) { memcpy(out, launches, (size_t)n_launches * sizeof launches[0]); return n_launches; }
int64_t fake_live(void) { return live; }
void fake_log(char *to, size_t room) { done = to; done_room = room; if (room) to[0] = 0; }
static void note(const char *what) {
    const size_t at = done ? strlen(done) : 0;
    if (done) snprintf(done + at, done_room - at, "%s %d, ", what, device);
}

int hipMalloc(void **p, size_t n) {
    *p = n <= malloc_limit ? calloc(1, n ? n : 1) : NULL;
    if (!*p) return last_error = OUT_OF_MEMORY;
    ++live;
    return OK;
}
int hipFree(void *p) { if (p) --live; free(p); return OK; }
int hipMemset(void *p, int v, size_t n) { memset(p, v, n); return OK; }
int hipMemcpy(void *d, const void *s, size_t n, int kind) { (void)kind; note("copy"); memcpy(d, s, n); return OK; }
int hipGetLastError(void) { const int e = last_error; last_error = OK; return e; }      /* reported once, as the runtime does */
int hipDeviceSynchronize(void) { note("sync"); return OK; }
int hipStreamSynchronize(void *s) { (void)s; return OK; }
int hipGetDevice(int *d) { *d = device; return OK; }
int hipSetDevice(int d) { device = d; return OK; }
int hipDeviceGetAttribute(int *v, int attr, int d) { (void)attr; (void)d; *v = cus; return OK; }
int hipGetDevicePropertiesR0600(void *p, int d) { (void)d; memset(p, 0, 1024); return OK; }     /* no number of CUs: the library takes 256 */
int hipGetSymbolAddress(void **p, const void *symbol) { *p = (void *)(uintptr_t)symbol; return OK; }
int hipFuncSetAttribute(const void *f, int attr, int v) { (void)f; (void)attr; (void)v; return OK; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int threads, size_t lds) {
    (void)f; (void)threads;
    *n = cu_lds && lds && cu_lds / lds < (size_t)resident ? (int)(cu_lds / lds) : resident;
    return OK;
}

static struct { dim3 grid, block; size_t lds; void *stream; } call;
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, void *stream) {
    call.grid = grid; call.block = block; call.lds = lds; call.stream = stream;
    return OK;
}
int __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, void **stream) {
    *grid = call.grid; *block = call.block; *lds = call.lds; *stream = call.stream;
    return OK;
}
int hipLaunchKernel(const void *f, dim3 grid, dim3 block, void **args, size_t lds, void *stream) {
    (void)f; (void)args; (void)stream;
    note("launch");
    if (n_launches < N_LAUNCHES) {
        uint32_t *l = launches[n_launches++];
        l[0] = grid.x; l[1] = grid.y; l[2] = block.x; l[3] = (uint32_t)lds;
    }
    return OK;
}
void **__hipRegisterFatBinary(const void *data) { static void *h; (void)data; return &h; }
void __hipUnregisterFatBinary(void **h) { (void)h; }
void __hipRegisterFunction(void **h, const void *f, char *df, const char *n, unsigned lim, void *a, void *b, void *c, void *d, int *w) {
    (void)h; (void)f; (void)df; (void)n; (void)lim; (void)a; (void)b; (void)c; (void)d; (void)w;
}
void __hipRegisterVar(void **h, void *v, char *hv, char *dv, int ext, size_t size, int constant, int global) {
    (void)h; (void)v; (void)hv; (void)dv; (void)ext; (void)size; (void)constant; (void)global;
}
