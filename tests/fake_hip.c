/* The HIP calls that libparquet makes, on the host: kernels are counted and not
 * run, device memory is host memory. Loaded globally before the library, so that
 * its calls come here (tests of the host code only). */
#include <pthread.h>
#include <stdlib.h>
#include <string.h>
#include <unistd.h>

typedef struct { unsigned x, y, z; } dim3;
typedef void* ptr;

int fake_host_fill = 0;                 /* byte that pinned memory starts with */
int fake_graph_us = 0;                  /* time spent in a graph call */
int fake_overlaps = 0;                  /* graph calls that met another thread's */
int fake_graph_calls = 0;
int fake_launches = 0;
unsigned fake_dims[4096][6];            /* grid and block of each launch */

static pthread_mutex_t mu = PTHREAD_MUTEX_INITIALIZER;
static pthread_t owner;
static int inside = 0;

static void enter(void) {
  pthread_mutex_lock(&mu);
  ++fake_graph_calls;
  if (inside && !pthread_equal(owner, pthread_self())) ++fake_overlaps;
  owner = pthread_self();
  ++inside;
  pthread_mutex_unlock(&mu);
  if (fake_graph_us) usleep(fake_graph_us);
}
static int leave(void) {
  pthread_mutex_lock(&mu);
  --inside;
  pthread_mutex_unlock(&mu);
  return 0;
}

int hipStreamBeginCapture(ptr s, int mode) { enter(); return 0; }
int hipStreamEndCapture(ptr s, ptr* g) { *g = (ptr)1; return leave(); }
int hipGraphInstantiate(ptr* e, ptr g, ptr* n, char* log, size_t size) { enter(); *e = (ptr)1; return leave(); }
int hipGraphLaunch(ptr e, ptr s) { enter(); return leave(); }
int hipGraphExecDestroy(ptr e) { enter(); return leave(); }
int hipGraphDestroy(ptr g) { enter(); return leave(); }

static __thread dim3 cfg_grid, cfg_block;
static __thread size_t cfg_shared;
static __thread ptr cfg_stream;
int __hipPushCallConfiguration(dim3 g, dim3 b, size_t sh, ptr s) {
  cfg_grid = g; cfg_block = b; cfg_shared = sh; cfg_stream = s;
  return 0;
}
int __hipPopCallConfiguration(dim3* g, dim3* b, size_t* sh, ptr* s) {
  *g = cfg_grid; *b = cfg_block; *sh = cfg_shared; *s = cfg_stream;
  return 0;
}
int hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t sh, ptr s) {
  pthread_mutex_lock(&mu);
  if (fake_launches < 4096) {
    const unsigned d[6] = {g.x, g.y, g.z, b.x, b.y, b.z};
    memcpy(fake_dims[fake_launches++], d, sizeof(d));
  }
  pthread_mutex_unlock(&mu);
  return 0;
}
int hipFuncSetAttribute(const void* f, int a, int v) { return 0; }

int hipHostMalloc(ptr* p, size_t n, unsigned flags) {
  *p = malloc(n);
  memset(*p, fake_host_fill, n);
  return 0;
}
int hipHostFree(ptr p) { free(p); return 0; }
int hipMemcpyAsync(ptr d, const void* s, size_t n, int kind, ptr st) { memmove(d, s, n); return 0; }
int hipMemsetAsync(ptr d, int v, size_t n, ptr s) { memset(d, v, n); return 0; }
int hipStreamSynchronize(ptr s) { return 0; }
int hipStreamCreateWithFlags(ptr* s, unsigned f) { *s = (ptr)2; return 0; }
int hipStreamDestroy(ptr s) { return 0; }
int hipStreamWaitEvent(ptr s, ptr e, unsigned f) { return 0; }
int hipEventCreate(ptr* e) { *e = (ptr)3; return 0; }
int hipEventCreateWithFlags(ptr* e, unsigned f) { *e = (ptr)3; return 0; }
int hipEventDestroy(ptr e) { return 0; }
int hipEventRecord(ptr e, ptr s) { return 0; }
int hipEventSynchronize(ptr e) { return 0; }
int hipEventElapsedTime(float* ms, ptr a, ptr b) { *ms = 1.0f; return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetLastError(void) { return 0; }
