/*
 * Stands in for the HIP runtime calls that libmeft makes, on a machine without a GPU: every launch, copy, event record and
 * stream wait is written to a list that a test reads back.  Loaded with RTLD_GLOBAL before the library.
 */
#define _GNU_SOURCE
#include <dlfcn.h>
#include <pthread.h>
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>
#include <string.h>
#include <unistd.h>

typedef struct { uint32_t x, y, z; } dim3_t;

typedef struct {
  char what[8];        /* launch, copy, record, wait */
  char name[256];      /* launch: the kernel's symbol */
  uint32_t grid[3], block[3];
  uint64_t lds;
  uint64_t stream, event, dst, src, bytes;
} rec_t;

#define CAP 4096
static rec_t recs[CAP];
static int n_recs;
static uint64_t next_handle = 0x1000;
static int32_t counts_value = 1;   /* what a copy to the host delivers in every word */

static int capturing;

/* rec_flip(n, f): another thread calls f(1) while the n-th launch from now on is under way; rec_flipped() waits for it */
static void (*flip_call)(int);
static int flip_in;
static pthread_t flip_thread;
static void* flip_main(void* arg) { (void)arg; flip_call(1); return NULL; }
void rec_flip(int n, void (*f)(int)) { flip_in = n; flip_call = f; }
int rec_flipped(void) {
  if (!flip_call || flip_in > 0) return 0;
  flip_call = NULL;
  return pthread_join(flip_thread, NULL) == 0;
}

void rec_capture(int on) { capturing = on; }
int rec_count(void) { return n_recs; }
const rec_t* rec_at(int i) { return &recs[i]; }
void rec_clear(void) { n_recs = 0; }

static rec_t* add(const char* what) {
  static rec_t spill;
  rec_t* r = n_recs < CAP ? &recs[n_recs++] : &spill;
  memset(r, 0, sizeof(*r));
  strncpy(r->what, what, sizeof(r->what) - 1);
  return r;
}

/* what a launch expression passes to the kernel's host stub */
static struct { dim3_t grid, block; size_t lds; void* stream; } config;
int __hipPushCallConfiguration(dim3_t grid, dim3_t block, size_t lds, void* stream) {
  config.grid = grid; config.block = block; config.lds = lds; config.stream = stream;
  return 0;
}
int __hipPopCallConfiguration(dim3_t* grid, dim3_t* block, size_t* lds, void** stream) {
  *grid = config.grid; *block = config.block; *lds = config.lds; *stream = config.stream;
  return 0;
}

int hipLaunchKernel(const void* f, dim3_t grid, dim3_t block, void** args, size_t lds, void* stream) {
  Dl_info info;
  rec_t* r = add("launch");
  (void)args;
  if (dladdr(f, &info) && info.dli_sname) strncpy(r->name, info.dli_sname, sizeof(r->name) - 1);
  r->grid[0] = grid.x; r->grid[1] = grid.y; r->grid[2] = grid.z;
  r->block[0] = block.x; r->block[1] = block.y; r->block[2] = block.z;
  r->lds = lds;
  r->stream = (uint64_t)(uintptr_t)stream;
  if (flip_in > 0 && --flip_in == 0) {
    if (pthread_create(&flip_thread, NULL, flip_main, NULL)) abort();
    usleep(100000);   /* a thread that does not have to wait for this call has come through by then */
  }
  return 0;
}

int hipMemcpyAsync(void* dst, const void* src, size_t bytes, int kind, void* stream) {
  rec_t* r = add("copy");
  r->dst = (uint64_t)(uintptr_t)dst; r->src = (uint64_t)(uintptr_t)src; r->bytes = bytes;
  r->stream = (uint64_t)(uintptr_t)stream;
  if (kind == 2) {   /* device to host: the counts the host waits for */
    int32_t* d = (int32_t*)dst;
    for (size_t i = 0; i < bytes / 4; ++i) d[i] = counts_value;
  }
  return 0;
}

static int handle(void** h) { *h = (void*)(uintptr_t)next_handle; next_handle += 0x100; return 0; }
int hipStreamCreateWithFlags(void** s, unsigned flags) { (void)flags; return handle(s); }
int hipEventCreateWithFlags(void** e, unsigned flags) { (void)flags; return handle(e); }
int hipEventCreate(void** e) { return handle(e); }
int hipEventDestroy(void* e) { (void)e; return 0; }
int hipEventSynchronize(void* e) { (void)e; return 0; }
int hipEventElapsedTime(float* ms, void* a, void* b) { (void)a; (void)b; *ms = 1.f; return 0; }
int hipEventRecord(void* e, void* stream) {
  rec_t* r = add("record");
  r->event = (uint64_t)(uintptr_t)e; r->stream = (uint64_t)(uintptr_t)stream;
  return 0;
}
int hipStreamWaitEvent(void* stream, void* e, unsigned flags) {
  rec_t* r = add("wait");
  (void)flags;
  r->event = (uint64_t)(uintptr_t)e; r->stream = (uint64_t)(uintptr_t)stream;
  return 0;
}
int hipStreamIsCapturing(void* stream, int* status) { (void)stream; *status = capturing; return 0; }
int hipHostMalloc(void** p, size_t bytes, unsigned flags) { (void)flags; *p = calloc(1, bytes); return *p ? 0 : 2; }
int hipFuncSetAttribute(const void* f, int attr, int value) { (void)f; (void)attr; (void)value; return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipGetSymbolAddress(void** p, const void* symbol) { (void)symbol; *p = (void*)0x100000; return 0; }
int hipGetLastError(void) { return 0; }
