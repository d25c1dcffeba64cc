/* Calls the library on the host with a stand-in for the parts of the HIP runtime it uses: memory
 * is the host's, launches and copies do nothing, and what the library asks the runtime for is
 * recorded.  (A program's own functions come before a shared library's of the same name.)
 *
 *   host_runtime page      a page of pinned memory can be had
 *   host_runtime nopage    it cannot
 *
 * Prints what was asked for, one "name value" per line. */
#include <pthread.h>
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#define __HIP_PLATFORM_AMD__ 1
#include <hip/hip_runtime_api.h>

#include "odb.h"

static int give_page;
static unsigned page_flags, event_flags;
static int pages, pages_freed, events, events_freed, event_waits, stream_waits, copies, launches;

hipError_t hipHostMalloc(void** p, size_t bytes, unsigned flags) {
    if (!give_page) return hipErrorOutOfMemory;
    page_flags = flags;
    pages += 1;
    *p = calloc(1, bytes);
    return *p ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipHostFree(void* p) {
    pages_freed += 1;
    free(p);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned flags) {
    event_flags = flags;
    events += 1;
    *e = (hipEvent_t)malloc(1);
    return hipSuccess;
}
hipError_t hipEventDestroy(hipEvent_t e) {
    events_freed += 1;
    free(e);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { return (void)e, (void)s, hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t e) { return (void)e, event_waits += 1, hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { return (void)s, stream_waits += 1, hipSuccess; }
hipError_t hipMemcpyAsync(void* dst, const void* src, size_t bytes, hipMemcpyKind kind, hipStream_t s) {
    (void)src, (void)kind, (void)s;
    memset(dst, 0, bytes);
    copies += 1;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 grid, dim3 block, void** args, size_t lds, hipStream_t s) {
    (void)f, (void)grid, (void)block, (void)args, (void)lds, (void)s;
    launches += 1;
    return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipGetDevice(int* dev) { return *dev = 0, hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int dev) {
    (void)a, (void)dev;
    return *v = 256, hipSuccess;
}

enum { kRank = 20000, kRanks = 2 };   /* ranks that take the path with a wait */

static void* calls(void* out) {
    static const int64_t off[kRanks + 1] = {0, kRank, 2 * kRank};
    static int64_t tok[1];   /* device pointers: never read here */
    static int32_t words[1];
    odb_window_t w = {kRanks, 0, 2 * kRank, off, tok, words, NULL, 0};
    const size_t bytes = odb_workspace_size(&w);
    void* ws = aligned_alloc(256, (bytes + 255) / 256 * 256);
    odb_length_sketch_t sk;
    int* st = out;
    st[0] = odb_form_groups(&w, 1000, words, words, words, words, ws, bytes, NULL);
    st[1] = odb_length_sketch(&w, NULL, 100, 1000, &sk, ws, bytes, NULL);
    st[2] = odb_form_groups(&w, 1000, words, words, words, words, ws, bytes, NULL);
    free(ws);
    return NULL;
}

int main(int argc, char** argv) {
    if (argc != 2) return 2;
    give_page = strcmp(argv[1], "page") == 0;
    int st[3] = {-1, -1, -1};
    pthread_t t;
    if (pthread_create(&t, NULL, calls, st) || pthread_join(t, NULL)) return 3;
    printf("status %d\n", st[0] | st[1] | st[2]);
    printf("pages %d\npages_freed %d\nevents %d\nevents_freed %d\n", pages, pages_freed, events, events_freed);
    printf("event_waits %d\nstream_waits %d\ncopies %d\nlaunches %d\n", event_waits, stream_waits, copies, launches);
    printf("page_coherent %d\npage_portable %d\n", (page_flags & hipHostMallocCoherent) != 0,
           (page_flags & hipHostMallocPortable) != 0);
    printf("event_untimed %d\n", (event_flags & hipEventDisableTiming) != 0);
    return 0;
}
