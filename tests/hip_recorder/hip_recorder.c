/*
 * A HIP runtime that runs nothing and writes down what it is asked for: the functions librb.so calls, loaded in front of the real
 * library by a process of its own (tests/recorded.py).  Streams, events and device memory are whatever numbers the caller uses.
 *
 * One line per stream operation: "launch KERNEL STREAM GRID BLOCK LDS [EVENT]" (EVENT: recorded by the launch's own completion),
 * "record EVENT STREAM", "wait STREAM EVENT", "sync STREAM".  Operations that were made to fail write nothing.
 */
#include <stdint.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef struct { uint32_t x, y, z; } dim3;
enum { OK = 0, INVALID_VALUE = 1, STREAM_CAPTURE_ISOLATION = 905 };

#define MAX_FUNCTIONS 4096
#define MAX_STREAMS 16
#define LOG_BYTES (1 << 20)

static struct { const void* host; const char* name; } functions[MAX_FUNCTIONS];
static int functions_known;
static char lines[LOG_BYTES];
static size_t used;
static int last_error;                  /* of any call, until it is asked for */
static char failing[64];                /* function whose calls fail, after so many that succeed */
static int failing_after;
static uintptr_t capturing[MAX_STREAMS], events_captured[64];
static uintptr_t events;                /* events are numbered from 1 */

#define WRITE(...) (used += (size_t)snprintf(lines + used, LOG_BYTES - used, __VA_ARGS__))

static int result(int e)
{
    if (e != OK) last_error = e;
    return e;
}

static int fails(const char* function)
{
    if (strcmp(failing, function) != 0) return 0;
    if (failing_after > 0) {
        --failing_after;
        return 0;
    }
    return 1;
}

static int is_capturing(uintptr_t stream)
{
    for (int i = 0; i < MAX_STREAMS; ++i)
        if (capturing[i] != 0 && capturing[i] == stream) return 1;
    return 0;
}

/* ---- for the test ---- */
const char* recorder_lines(void) { return lines; }
void recorder_clear(void) { used = 0; lines[0] = 0; }
void recorder_fail(const char* function, int after) { snprintf(failing, sizeof failing, "%s", function); failing_after = after; }
void recorder_pend(int error) { last_error = error; }
int recorder_pending(void) { return last_error; }
void recorder_capture(uintptr_t stream)
{
    for (int i = 0; i < MAX_STREAMS; ++i)
        if (capturing[i] == 0) { capturing[i] = stream; return; }
}
void recorder_end_capture(void) { memset(capturing, 0, sizeof capturing); }

/* ---- the code object ---- */
void** __hipRegisterFatBinary(const void* data) { (void)data; static void* module; return &module; }
void __hipUnregisterFatBinary(void** module) { (void)module; }
void __hipRegisterVar(void) {}
void __hipRegisterFunction(void** module, const void* host, char* device, const char* name)
{
    (void)module; (void)device;
    if (functions_known == MAX_FUNCTIONS) abort();
    functions[functions_known].host = host;
    functions[functions_known++].name = name;
}

/* ---- launches ---- */
static struct { dim3 grid, block; size_t lds; uintptr_t stream; } pushed;
int __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, uintptr_t stream)
{
    pushed.grid = grid; pushed.block = block; pushed.lds = lds; pushed.stream = stream;
    return OK;
}
int __hipPopCallConfiguration(dim3* grid, dim3* block, size_t* lds, uintptr_t* stream)
{
    *grid = pushed.grid; *block = pushed.block; *lds = pushed.lds; *stream = pushed.stream;
    return OK;
}

static void launched(const void* host, dim3 grid, dim3 block, size_t lds, uintptr_t stream)
{
    const char* name = "?";
    for (int i = 0; i < functions_known; ++i)
        if (functions[i].host == host) name = functions[i].name;
    WRITE("launch %s %ju %u %u %zu", name, (uintmax_t)stream, grid.x, block.x, lds);
}

int hipLaunchKernel(const void* host, dim3 grid, dim3 block, void** args, size_t lds, uintptr_t stream)
{
    (void)args;
    if (fails("hipLaunchKernel")) return result(INVALID_VALUE);
    launched(host, grid, block, lds, stream);
    WRITE("\n");
    return OK;
}

int hipExtLaunchKernel(const void* host, dim3 grid, dim3 block, void** args, size_t lds, uintptr_t stream, uintptr_t start, uintptr_t stop, int flags)
{
    (void)args; (void)flags;
    if (start != 0 || is_capturing(stream) || fails("hipExtLaunchKernel")) return result(INVALID_VALUE);
    launched(host, grid, block, lds, stream);
    WRITE(" %ju\n", (uintmax_t)stop);
    events_captured[stop] = 0;
    return OK;
}

/* ---- streams and events ---- */
int hipEventCreateWithFlags(uintptr_t* event, unsigned flags)
{
    (void)flags;
    if (events + 1 == 64) abort();
    *event = ++events;
    return OK;
}
int hipEventDestroy(uintptr_t event) { (void)event; return OK; }

int hipEventRecord(uintptr_t event, uintptr_t stream)
{
    if (fails("hipEventRecord")) return result(INVALID_VALUE);
    events_captured[event] = (uintptr_t)is_capturing(stream);
    WRITE("record %ju %ju\n", (uintmax_t)event, (uintmax_t)stream);
    return OK;
}

int hipStreamWaitEvent(uintptr_t stream, uintptr_t event, unsigned flags)
{
    (void)flags;
    if (fails("hipStreamWaitEvent")) return result(INVALID_VALUE);
    if (is_capturing(stream) && !events_captured[event]) return result(STREAM_CAPTURE_ISOLATION);
    if (!is_capturing(stream) && events_captured[event]) recorder_capture(stream);       /* joins the capture */
    WRITE("wait %ju %ju\n", (uintmax_t)stream, (uintmax_t)event);
    return OK;
}

int hipStreamIsCapturing(uintptr_t stream, int* status)
{
    if (fails("hipStreamIsCapturing")) return result(INVALID_VALUE);
    *status = is_capturing(stream);
    return OK;
}

int hipStreamSynchronize(uintptr_t stream) { WRITE("sync %ju\n", (uintmax_t)stream); return OK; }

/* ---- the rest ---- */
int hipGetLastError(void)
{
    const int e = last_error;
    last_error = OK;
    return e;
}
int hipGetDevice(int* device) { *device = 0; return OK; }
int hipFuncSetAttribute(const void* host, int attribute, int value) { (void)host; (void)attribute; (void)value; return OK; }
int hipGetSymbolAddress(void** p, const void* symbol) { (void)symbol; *p = NULL; return result(INVALID_VALUE); }
int hipMemcpy(void* to, const void* from, size_t bytes, int kind) { (void)from; (void)kind; memset(to, 0, bytes); return OK; }
int hipPointerGetAttributes(void* attributes, const void* p) { (void)attributes; (void)p; return result(INVALID_VALUE); }
