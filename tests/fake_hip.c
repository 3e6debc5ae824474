/* Host stand-in for the HIP calls of libtau1.so: device memory is host memory,
 * kernels do nothing, and the calls that the tests ask about are counted.
 * Loaded with RTLD_GLOBAL before the library, in a process of its own. */
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
#include <pthread.h>

enum { OK = 0, OUT_OF_MEMORY = 2, CAPTURING = 900 };

unsigned fake_pinned_flags, fake_event_flags;
int fake_grid;                     /* workgroups of the last launch */
int fake_launches, fake_graph_builds, fake_graph_nodes, fake_events, fake_pinned, fake_copies;
int fake_freed_here, fake_freed;   /* hipHostFree: on the main thread, on any */
int fake_refuse_pinned, fake_capturing;
#define INC(c) __atomic_add_fetch(&(c), 1, __ATOMIC_SEQ_CST)   /* calls come from several threads */
static pthread_t main_thread;

__attribute__((constructor)) static void init(void) { main_thread = pthread_self(); }

int hipGetDevice(int *d) { *d = 0; return OK; }
int hipGetLastError(void) { return OK; }
int hipGetSymbolAddress(void **p, const void *s) { (void)s; *p = NULL; return 1; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int b, size_t l) {
    (void)f; (void)b; (void)l;
    *n = 2;
    return OK;
}
int hipHostMalloc(void **p, size_t n, unsigned flags) {
    fake_pinned_flags = flags;
    if (fake_refuse_pinned) return OUT_OF_MEMORY;
    INC(fake_pinned);
    *p = calloc(1, n);
    return OK;
}
int hipHostFree(void *p) {
    if (pthread_equal(pthread_self(), main_thread)) INC(fake_freed_here);
    INC(fake_freed);
    free(p);
    return OK;
}
int hipEventCreate(void **e) { *e = malloc(1); return OK; }
int hipEventCreateWithFlags(void **e, unsigned flags) {
    fake_event_flags = flags;
    INC(fake_events);
    *e = malloc(1);
    return OK;
}
int hipEventDestroy(void *e) { free(e); return OK; }
int hipEventRecord(void *e, void *s) { (void)e; (void)s; return OK; }
int hipEventSynchronize(void *e) { (void)e; return fake_capturing ? CAPTURING : OK; }
int hipEventElapsedTime(float *ms, void *a, void *b) { (void)a; (void)b; *ms = 1.0f; return OK; }
int hipStreamSynchronize(void *s) { (void)s; return fake_capturing ? CAPTURING : OK; }
int hipStreamIsCapturing(void *s, int *st) { (void)s; *st = fake_capturing; return OK; }
int hipThreadExchangeStreamCaptureMode(int *m) { *m = 0; return OK; }
int hipMemcpyAsync(void *d, const void *s, size_t n, int kind, void *st) {
    (void)kind; (void)st;
    INC(fake_copies);
    memcpy(d, s, n);
    return OK;
}
int hipMemsetAsync(void *d, int v, size_t n, void *st) { (void)st; memset(d, v, n); return OK; }
typedef struct { unsigned x, y, z; } dim3_t;
int __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t l, void *s) {
    (void)g; (void)b; (void)l; (void)s;
    return OK;
}
int __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *l, void **s) {
    *g = *b = (dim3_t){1, 1, 1};
    *l = 0;
    *s = NULL;
    return OK;
}
int hipLaunchKernel(const void *f, dim3_t g, dim3_t b, void **a, size_t l, void *s) {
    (void)f; (void)b; (void)a; (void)l; (void)s;
    fake_grid = (int)g.x;
    INC(fake_launches);
    return OK;
}
int hipGraphCreate(void **g, unsigned f) { (void)f; *g = malloc(1); return OK; }
int hipGraphDestroy(void *g) { free(g); return OK; }
int hipGraphAddKernelNode(void **n, void *g, const void *d, size_t k, const void *p) {
    (void)g; (void)d; (void)k; (void)p;
    INC(fake_graph_nodes);
    *n = (void *)(uintptr_t)fake_graph_nodes;
    return OK;
}
int hipGraphInstantiate(void **e, void *g, void *n, char *l, size_t s) {
    (void)g; (void)n; (void)l; (void)s;
    INC(fake_graph_builds);
    *e = malloc(1);
    return OK;
}
int hipGraphExecDestroy(void *e) { free(e); return OK; }
int hipGraphLaunch(void *e, void *s) { (void)e; (void)s; return OK; }
