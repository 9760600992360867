/* A stand-in for the HIP runtime, for host tests of the library's own
 * bookkeeping (libpet_os.so resolves its HIP calls to the test program):
 * device memory is host memory, kernels do nothing, and the work of a stream
 * stays pending until the host waits for it or the test says that it is done. */
#ifndef HIP_STUB_H
#define HIP_STUB_H
#include <stddef.h>

extern long stub_mallocs, stub_frees;        /* allocations made, memory given back */
extern size_t stub_live, stub_limit;         /* bytes allocated; above stub_limit hipMalloc fails */
extern long stub_host_waits;                 /* host waits that found pending work */
extern long stub_stream_waits;               /* hipStreamWaitEvent for an event that is pending on another stream */
extern long stub_launches;                   /* kernels launched */
extern long stub_fail_launch;                /* the launch of this number fails (-1: none) */
extern int stub_capturing;                   /* another stream of this thread captures (global mode) */
extern long stub_capture_breaks;             /* calls that would have broken that capture */
extern void* stub_last_copy;                 /* device side of the last hipMemcpyAsync */
extern void* stub_last_malloc;               /* the last allocation */
extern void (*stub_on_wait)(void);           /* called inside a host wait for pending work */

void stub_finish(void* stream);              /* the stream's work is done */
int stub_pending(void* stream);
void* stub_block(const void* p);             /* base of the allocation that holds p (null: none) */
size_t stub_block_bytes(const void* p);
int stub_launches_of(const char* kernel);    /* launches of kernels whose name holds this text */
#endif
