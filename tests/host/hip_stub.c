#include "hip_stub.h"

#include <pthread.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

enum { OK = 0, INVALID = 1, OOM = 2, NOT_READY = 600, CAPTURE = 900, LAUNCH = 719 };

long stub_mallocs, stub_frees, stub_host_waits, stub_stream_waits, stub_launches, stub_capture_breaks;
long stub_fail_launch = -1;
size_t stub_live, stub_limit = (size_t)1 << 34;
int stub_capturing;
void *stub_last_copy, *stub_last_malloc;
void (*stub_on_wait)(void);

static pthread_mutex_t mu = PTHREAD_MUTEX_INITIALIZER;
static __thread int relaxed, last_error;

/* streams: work queued and done (counts), and what another stream's work waits for */
typedef struct Stream { void* s; long queued, done; struct { struct Stream* on; long at; } dep[64]; int n_dep; } Stream;
static Stream streams[64];
static int n_streams;
static Stream* stream_of(void* s) {
    for (int k = 0; k < n_streams; ++k)
        if (streams[k].s == s) return &streams[k];
    streams[n_streams].s = s;
    return &streams[n_streams++];
}
static void done_to(Stream* S, long at) {
    if (S->done >= at) return;
    S->done = at;
    for (int k = 0; k < S->n_dep; ++k) done_to(S->dep[k].on, S->dep[k].at);
    S->n_dep = 0;
}
void stub_finish(void* s) {
    pthread_mutex_lock(&mu);
    Stream* S = stream_of(s);
    done_to(S, S->queued);
    pthread_mutex_unlock(&mu);
}
int stub_pending(void* s) {
    pthread_mutex_lock(&mu);
    Stream* S = stream_of(s);
    int p = S->done < S->queued;
    pthread_mutex_unlock(&mu);
    return p;
}
static int fin(int e) {
    if (e) last_error = e;
    return e;
}
/* a call that may not be made while a stream of the thread captures */
static int unsafe(void) {
    if (!stub_capturing || relaxed) return 0;
    ++stub_capture_breaks;
    return 1;
}
static void host_wait(Stream* S) {
    if (S->done >= S->queued) return;
    ++stub_host_waits;
    if (stub_on_wait) {
        pthread_mutex_unlock(&mu);
        stub_on_wait();
        pthread_mutex_lock(&mu);
    }
    done_to(S, S->queued);
}

/* memory */
typedef struct { char* p; size_t n; } Block;
static Block blocks[4096];
static int n_blocks;
int hipMalloc(void** p, size_t n) {
    if (unsafe()) return fin(CAPTURE);
    pthread_mutex_lock(&mu);
    int rc = OOM;
    if (stub_live + n <= stub_limit) {
        char* q = calloc(1, n ? n : 1);
        blocks[n_blocks++] = (Block){q, n};
        stub_live += n;
        ++stub_mallocs;
        stub_last_malloc = q;
        *p = q;
        rc = OK;
    }
    pthread_mutex_unlock(&mu);
    return fin(rc);
}
int hipFree(void* p) {
    if (unsafe()) return fin(CAPTURE);
    if (!p) return OK;
    pthread_mutex_lock(&mu);
    for (int k = 0; k < n_streams; ++k) host_wait(&streams[k]);
    int rc = INVALID;
    for (int k = 0; k < n_blocks; ++k)
        if (blocks[k].p == p) {
            stub_live -= blocks[k].n;
            ++stub_frees;
            free(p);
            blocks[k] = blocks[--n_blocks];
            rc = OK;
            break;
        }
    pthread_mutex_unlock(&mu);
    return fin(rc);
}
static Block* block_of(const void* p) {
    for (int k = 0; k < n_blocks; ++k)
        if ((char*)p >= blocks[k].p && (char*)p < blocks[k].p + blocks[k].n) return &blocks[k];
    return NULL;
}
void* stub_block(const void* p) {
    Block* b = block_of(p);
    return b ? b->p : NULL;
}
size_t stub_block_bytes(const void* p) {
    Block* b = block_of(p);
    return b ? b->n : 0;
}
int hipMemcpy(void* d, const void* s, size_t n, int kind) {
    (void)kind;
    memcpy(d, s, n);
    return OK;
}
int hipMemcpyAsync(void* d, const void* s, size_t n, int kind, void* st) {
    memcpy(d, s, n);
    pthread_mutex_lock(&mu);
    stub_last_copy = (void*)(kind == 1 ? d : s);
    stream_of(st)->queued++;
    pthread_mutex_unlock(&mu);
    return OK;
}
int hipMemset(void* p, int v, size_t n) {
    memset(p, v, n);
    return OK;
}
int hipGetSymbolAddress(void** p, const void* s) {
    (void)s;
    static char* area;
    if (!area) area = calloc(1, (size_t)256 << 20);
    *p = area;
    return OK;
}

/* events */
typedef struct { void* s; long at; int recorded; } Event;
int hipEventCreateWithFlags(void** e, unsigned f) {
    (void)f;
    *e = calloc(1, sizeof(Event));
    return OK;
}
int hipEventCreate(void** e) { return hipEventCreateWithFlags(e, 0); }
int hipEventDestroy(void* e) {
    free(e);
    return OK;
}
int hipEventRecord(void* e, void* s) {
    pthread_mutex_lock(&mu);
    Stream* S = stream_of(s);
    *(Event*)e = (Event){s, S->queued, 1};
    pthread_mutex_unlock(&mu);
    return OK;
}
static int event_pending(Event* e) { return e->recorded && stream_of(e->s)->done < e->at; }
int hipEventQuery(void* e) {
    if (unsafe()) return fin(CAPTURE);
    pthread_mutex_lock(&mu);
    int p = event_pending(e);
    pthread_mutex_unlock(&mu);
    return p ? NOT_READY : OK;
}
int hipEventSynchronize(void* e) {
    if (unsafe()) return fin(CAPTURE);
    pthread_mutex_lock(&mu);
    if (event_pending(e)) host_wait(stream_of(((Event*)e)->s));
    pthread_mutex_unlock(&mu);
    return OK;
}
int hipEventElapsedTime(float* ms, void* a, void* b) {
    (void)a;
    (void)b;
    *ms = 1.0f;
    return OK;
}

/* streams */
int hipStreamWaitEvent(void* s, void* e, unsigned f) {
    (void)f;
    pthread_mutex_lock(&mu);
    Event* E = e;
    if (event_pending(E) && E->s != s) {
        ++stub_stream_waits;
        Stream* S = stream_of(s);
        S->queued++;
        S->dep[S->n_dep].on = stream_of(E->s);
        S->dep[S->n_dep++].at = E->at;
    }
    pthread_mutex_unlock(&mu);
    return OK;
}
int hipStreamSynchronize(void* s) {
    if (unsafe()) return fin(CAPTURE);
    pthread_mutex_lock(&mu);
    host_wait(stream_of(s));
    pthread_mutex_unlock(&mu);
    return OK;
}
int hipDeviceSynchronize(void) {
    if (unsafe()) return fin(CAPTURE);
    pthread_mutex_lock(&mu);
    for (int k = 0; k < n_streams; ++k) host_wait(&streams[k]);
    pthread_mutex_unlock(&mu);
    return OK;
}
int hipStreamCreateWithFlags(void** s, unsigned f) {
    (void)f;
    *s = calloc(1, 16);
    return OK;
}
int hipStreamDestroy(void* s) {
    (void)s;
    return OK;
}
int hipStreamIsCapturing(void* s, int* status) {
    (void)s;
    *status = 0;
    return OK;
}
int hipThreadExchangeStreamCaptureMode(int* mode) {
    int was = relaxed ? 2 : 0;
    relaxed = *mode == 2;
    *mode = was;
    return OK;
}

/* device, errors */
int hipGetDevice(int* d) {
    *d = 0;
    return OK;
}
int hipSetDevice(int d) {
    (void)d;
    return OK;
}
int hipGetLastError(void) {
    int e = last_error;
    last_error = 0;
    return e;
}
const char* hipGetErrorString(int e) {
    (void)e;
    return "stub error";
}

/* kernels */
static struct { const void* f; char name[256]; int n; } kernels[512];
static int n_kernels;
void** __hipRegisterFatBinary(const void* d) {
    (void)d;
    static void* h[1];
    return h;
}
void __hipUnregisterFatBinary(void** h) { (void)h; }
void __hipRegisterFunction(void** h, const void* f, char* dn, const char* name, unsigned l, void* a, void* b, void* c,
                           void* d, int* w) {
    (void)h, (void)dn, (void)l, (void)a, (void)b, (void)c, (void)d, (void)w;
    kernels[n_kernels].f = f;
    snprintf(kernels[n_kernels++].name, sizeof(kernels[0].name), "%s", name);
}
void __hipRegisterVar(void** h, void* v, char* a, char* b, int c, size_t n, int d, int e) {
    (void)h, (void)v, (void)a, (void)b, (void)c, (void)n, (void)d, (void)e;
}
typedef struct { unsigned x, y, z; } Dim3;
static __thread struct { Dim3 g, b; size_t n; void* s; } cfg;
int __hipPushCallConfiguration(Dim3 g, Dim3 b, size_t n, void* s) {
    cfg.g = g;
    cfg.b = b;
    cfg.n = n;
    cfg.s = s;
    return OK;
}
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* n, void** s) {
    *g = cfg.g;
    *b = cfg.b;
    *n = cfg.n;
    *s = cfg.s;
    return OK;
}
int hipLaunchKernel(const void* f, Dim3 g, Dim3 b, void** args, size_t n, void* s) {
    (void)args, (void)n;
    pthread_mutex_lock(&mu);
    int bad = stub_launches++ == stub_fail_launch;
    /* the limits of a launch */
    if (!g.x || !g.y || !g.z || g.y > 65535 || g.z > 65535 || (uint64_t)g.x * b.x >= (1ull << 32) ||
        (uint64_t)g.y * b.y >= (1ull << 32) || (uint64_t)g.z * b.z >= (1ull << 32))
        bad = 1;
    if (!bad) {
        stream_of(s)->queued++;
        for (int k = 0; k < n_kernels; ++k)
            if (kernels[k].f == f) kernels[k].n++;
    }
    pthread_mutex_unlock(&mu);
    return fin(bad ? LAUNCH : OK);
}
int hipExtLaunchKernel(const void* f, Dim3 g, Dim3 b, void** args, size_t n, void* s, void* e0, void* e1, int fl) {
    (void)e0, (void)e1, (void)fl;
    return hipLaunchKernel(f, g, b, args, n, s);
}
int stub_launches_of(const char* name) {
    int n = 0;
    for (int k = 0; k < n_kernels; ++k)
        if (strstr(kernels[k].name, name)) n += kernels[k].n;
    return n;
}
