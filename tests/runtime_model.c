/* A model of the HIP runtime for tests on a machine without a GPU: the calls
 * the library makes, with the lifetimes of what they are given.  Streams queue
 * copies, launches, event records and graph replays and run them when something
 * waits for them; handles and memory are checked at every use.  Misuse is
 * counted under a name (model_violations); model_fail_at(n) makes the n-th call
 * from now that can fail do so. */
#define _GNU_SOURCE
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

typedef int E;
typedef struct { unsigned x, y, z; } dim3_t;
enum { kOk = 0, kErr = 999 };

/* ---- objects */
typedef enum { kMem, kPinned, kStream, kEvent, kGraph, kExec } Kind;
typedef struct Obj {
    Kind kind;
    int live, capturing, bad_capture;
    long pending;             /* queued operations that use it */
    char *ptr;
    size_t bytes;
    struct Obj *next;
} Obj;
static Obj *objs;
static Obj null_stream = {kStream, 1, 0, 0, 0, NULL, 0, NULL};

static char log_[1 << 14];
static long violations, calls, fail_at, syncs, copies, launches, replays;
static E last_error;

static void bad(const char *what)
{
    ++violations;
    if (strlen(log_) + strlen(what) + 2 < sizeof log_) strcat(strcat(log_, what), "\n");
}

static Obj *make(Kind k)
{
    Obj *o = calloc(1, sizeof *o);   /* never freed: a stale handle stays recognisable */
    o->kind = k;
    o->live = 1;
    o->next = objs;
    return objs = o;
}

static Obj *use(void *h, Kind k, const char *who)
{
    if (k == kStream && !h) return &null_stream;
    for (Obj *o = objs; o; o = o->next)
        if (o == h) {
            if (o->kind != k || !o->live) bad(who);
            return o;
        }
    bad(who);
    return NULL;
}

static Obj *memory(const void *p, size_t n, const char *who)
{
    for (Obj *o = objs; o; o = o->next)
        if ((o->kind == kMem || o->kind == kPinned) && o->live && (const char *)p >= o->ptr &&
            (const char *)p + n <= o->ptr + o->bytes)
            return o;
    bad(who);
    return NULL;
}

/* ---- queued work: one list over all streams, in issue order */
typedef struct Op {
    Obj *stream, *event, *exec, *dst, *src;
    char *to;
    const char *from;
    size_t n;
    int done;
    struct Op *next;
} Op;
static Op *ops;

static void enqueue(Op o)
{
    Op **p = &ops;
    while (*p) p = &(*p)->next;
    *p = malloc(sizeof o);
    **p = o;
    (*p)->next = NULL;
    Obj *held[] = {o.stream, o.event, o.exec, o.dst, o.src};
    for (int i = 0; i < 5; ++i)
        if (held[i]) ++held[i]->pending;
}

/* runs what is queued, of one stream or (null) of all, up to an operation */
static void run(Obj *stream, const Op *upto)
{
    for (Op **p = &ops; *p;) {
        Op *o = *p;
        if (stream && o->stream != stream) {
            p = &o->next;
            continue;
        }
        if (o->n) memcpy(o->to, o->from, o->n);
        Obj *held[] = {o->stream, o->event, o->exec, o->dst, o->src};
        for (int i = 0; i < 5; ++i)
            if (held[i]) --held[i]->pending;
        const int last = o == upto;
        *p = o->next;
        free(o);
        if (last) return;
    }
}

static int fails(void)
{
    ++calls;
    if (fail_at > 0 && --fail_at == 0) {
        last_error = kErr;
        return 1;
    }
    return 0;
}

/* ---- what the tests ask */
long model_violations(char *text, size_t n)
{
    if (n) {
        strncpy(text, log_, n - 1);
        text[n - 1] = 0;
    }
    return violations;
}
void model_fail_at(long n) { fail_at = n; }
long model_calls(void) { return calls; }
long model_syncs(void) { return syncs; }
long model_copies(void) { return copies; }
long model_launches(void) { return launches; }
long model_replays(void) { return replays; }
long model_live(void)
{
    long n = 0;
    for (Obj *o = objs; o; o = o->next) n += o->live;
    return n;
}

/* ---- the runtime */
static E alloc(void **p, size_t n, Kind k)
{
    if (fails()) return kErr;
    Obj *o = make(k);
    o->bytes = n;
    o->ptr = aligned_alloc(256, (n + 255) / 256 * 256);
    memset(o->ptr, 0xa5, n);
    *p = o->ptr;
    return kOk;
}
static E release(void *p, Kind k, const char *who)
{
    if (!p) return kOk;
    for (Obj *o = objs; o; o = o->next)
        if (o->kind == k && o->live && o->ptr == p) {
            if (o->pending) bad(who);
            o->live = 0;
            free(o->ptr);
            o->ptr = NULL;
            o->bytes = 0;
            return kOk;
        }
    bad(who);
    return kErr;
}
E hipMalloc(void **p, size_t n) { return alloc(p, n, kMem); }
E hipHostMalloc(void **p, size_t n, unsigned f) { (void)f; return alloc(p, n, kPinned); }
E hipFree(void *p) { return release(p, kMem, "hipFree: unknown or in use"); }
E hipHostFree(void *p) { return release(p, kPinned, "hipHostFree: unknown or in use"); }
E hipMemset(void *d, int v, size_t n) { if (fails()) return kErr; run(NULL, NULL); memory(d, n, "hipMemset"); memset(d, v, n); return kOk; }
E hipMemsetAsync(void *d, int v, size_t n, void *s) { (void)s; return hipMemset(d, v, n); }
E hipMemcpyAsync(void *d, const void *s, size_t n, int k, void *st)
{
    (void)k;
    if (fails()) return kErr;
    ++copies;
    Obj *q = use(st, kStream, "hipMemcpyAsync: stream");
    if (q && q->capturing) {
        q->bad_capture = 1;
        return kErr;
    }
    Op o = {.stream = q, .to = d, .from = s, .n = n};
    o.dst = memory(d, n, "hipMemcpyAsync: destination");
    o.src = memory(s, n, "hipMemcpyAsync: source");
    enqueue(o);
    return kOk;
}
E hipDeviceSynchronize(void) { if (fails()) return kErr; ++syncs; run(NULL, NULL); return kOk; }
E hipStreamSynchronize(void *s) { if (fails()) return kErr; run(use(s, kStream, "hipStreamSynchronize"), NULL); return kOk; }
E hipStreamCreateWithFlags(void **s, unsigned f) { (void)f; if (fails()) return kErr; *s = make(kStream); return kOk; }
E hipStreamDestroy(void *s)
{
    Obj *o = use(s, kStream, "hipStreamDestroy");
    if (!o || o == &null_stream) return kErr;
    if (o->pending) bad("hipStreamDestroy: work is queued");
    o->live = 0;
    return kOk;
}
E hipStreamWaitEvent(void *s, void *e, unsigned f)
{
    (void)f;
    if (fails()) return kErr;
    Obj *q = use(s, kStream, "hipStreamWaitEvent: stream"), *v = use(e, kEvent, "hipStreamWaitEvent: event");
    if (q && v && v->capturing) q->capturing = 1;
    return kOk;
}
E hipStreamIsCapturing(void *s, int *c) { Obj *o = use(s, kStream, "hipStreamIsCapturing"); *c = o ? o->capturing : 0; return kOk; }
E hipStreamBeginCapture(void *s, int m)
{
    (void)m;
    if (fails()) return kErr;
    Obj *o = use(s, kStream, "hipStreamBeginCapture");
    if (o->capturing) bad("hipStreamBeginCapture: capturing already");
    o->capturing = 1;
    o->bad_capture = 0;
    return kOk;
}
E hipStreamEndCapture(void *s, void **g)
{
    Obj *o = use(s, kStream, "hipStreamEndCapture");
    if (!o->capturing) bad("hipStreamEndCapture: not capturing");
    const int failed = o->bad_capture;
    for (Obj *q = objs; q; q = q->next)
        if (q->kind == kStream || q->kind == kEvent) q->capturing = 0;
    if (fails() || failed) return kErr;
    *g = make(kGraph);
    return kOk;
}
E hipEventCreateWithFlags(void **e, unsigned f) { (void)f; if (fails()) return kErr; *e = make(kEvent); return kOk; }
E hipEventCreate(void **e) { return hipEventCreateWithFlags(e, 0); }
E hipEventDestroy(void *e)
{
    Obj *o = use(e, kEvent, "hipEventDestroy");
    if (!o) return kErr;
    if (o->pending) bad("hipEventDestroy: a record is queued");
    o->live = 0;
    return kOk;
}
E hipEventRecord(void *e, void *s)
{
    if (fails()) return kErr;
    Obj *v = use(e, kEvent, "hipEventRecord: event"), *q = use(s, kStream, "hipEventRecord: stream");
    if (!v || !q) return kErr;
    v->capturing = q->capturing;
    if (!q->capturing) {
        Op o = {.stream = q, .event = v};
        enqueue(o);
    }
    return kOk;
}
E hipEventSynchronize(void *e)
{
    if (fails()) return kErr;
    Obj *v = use(e, kEvent, "hipEventSynchronize");
    const Op *last = NULL;
    for (const Op *o = ops; o; o = o->next)
        if (o->event == v) last = o;
    if (last) run(last->stream, last);
    return kOk;
}
E hipEventElapsedTime(float *t, void *a, void *b)
{
    use(a, kEvent, "hipEventElapsedTime");
    use(b, kEvent, "hipEventElapsedTime");
    *t = 1.f;
    return kOk;
}
E hipGraphInstantiate(void **x, void *g, void *n, char *c, size_t s)
{
    (void)n; (void)c; (void)s;
    if (fails()) return kErr;
    use(g, kGraph, "hipGraphInstantiate");
    *x = make(kExec);
    return kOk;
}
E hipGraphLaunch(void *x, void *s)
{
    if (fails()) return kErr;
    ++replays;
    Op o = {.stream = use(s, kStream, "hipGraphLaunch: stream"), .exec = use(x, kExec, "hipGraphLaunch")};
    enqueue(o);
    return kOk;
}
E hipGraphDestroy(void *g) { Obj *o = use(g, kGraph, "hipGraphDestroy"); if (o) o->live = 0; return kOk; }
E hipGraphExecDestroy(void *x)
{
    Obj *o = use(x, kExec, "hipGraphExecDestroy");
    if (!o) return kErr;
    if (o->pending) bad("hipGraphExecDestroy: a replay is queued");
    o->live = 0;
    return kOk;
}
E hipLaunchKernel(const void *f, dim3_t g, dim3_t b, void **args, size_t l, void *s)
{
    (void)f; (void)g; (void)b; (void)args; (void)l;
    if (fails()) return kErr;
    ++launches;
    Obj *q = use(s, kStream, "hipLaunchKernel: stream");
    if (q && !q->capturing) {
        Op o = {.stream = q};
        enqueue(o);
    }
    return kOk;
}
E hipDeviceGetAttribute(int *v, int a, int d) { (void)a; (void)d; *v = 256; return kOk; }
E hipFuncSetAttribute(const void *f, int a, int v) { (void)f; (void)a; (void)v; return fails() ? kErr : kOk; }
E hipGetDevice(int *d) { *d = 0; return kOk; }
E hipGetDeviceCount(int *n) { *n = 1; return kOk; }
E hipSetDevice(int d) { (void)d; return kOk; }
E hipGetLastError(void) { const E e = last_error; last_error = kOk; return e; }
E hipGetSymbolAddress(void **p, const void *s) { (void)s; return hipMalloc(p, 16 << 20); }
E hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *f, int t, size_t l) { (void)f; (void)t; (void)l; *n = 1; return kOk; }

/* ---- kernel registration and launch configuration */
static dim3_t cfg_grid, cfg_block;
static size_t cfg_lds;
static void *cfg_stream;
E __hipPushCallConfiguration(dim3_t g, dim3_t b, size_t l, void *s) { cfg_grid = g; cfg_block = b; cfg_lds = l; cfg_stream = s; return kOk; }
E __hipPopCallConfiguration(dim3_t *g, dim3_t *b, size_t *l, void **s) { *g = cfg_grid; *b = cfg_block; *l = cfg_lds; *s = cfg_stream; return kOk; }
void **__hipRegisterFatBinary(const void *d) { static void *h; (void)d; return &h; }
void __hipUnregisterFatBinary(void **m) { (void)m; }
void __hipRegisterFunction(void **m, const void *h, char *d, const char *n, unsigned t, void *a, void *b, void *c, void *e, int *w)
{
    (void)m; (void)h; (void)d; (void)n; (void)t; (void)a; (void)b; (void)c; (void)e; (void)w;
}
void __hipRegisterVar(void **m, void *v, char *h, char *n, int e, size_t s, int c, int g)
{
    (void)m; (void)v; (void)h; (void)n; (void)e; (void)s; (void)c; (void)g;
}
