// runtime_check.cpp -- drives the host runtime (csrc/runtime.cpp,
// csrc/noalloc.cpp and csrc/server.cpp) on the CPU, over a stand-in for the HIP runtime: device
// memory is host memory, streams run at once, and the kernels' launches are
// recorded and do nothing (a selection reports the totals set here).  So it
// shows what the host code allocates, captures, launches and refuses.
//   runtime_check dense     a DENSE view whose staging is gone is refused
//   runtime_check graph     a captured graph is replayed while its capacities hold
//   runtime_check server    restores beside a checkpoint; finishes through staging
//   runtime_check link      what kernels read and write over the host link
//   runtime_check capture   what an allocation-free call puts into a capture
// Exit status 0 when every check holds; the first failing check is printed.
#include <algorithm>
#include <chrono>
#include <condition_variable>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "ckpt.h"
#include "ckpt_runtime.h"

using namespace ckpt;

#define CHECK(cond)                                                                  \
    do {                                                                             \
        if (!(cond)) {                                                               \
            printf("line %d: %s (%s)\n", __LINE__, #cond, ckpt_last_error());        \
            exit(1);                                                                 \
        }                                                                            \
    } while (0)

// ------------------------------------------------- stand-in for HIP runtime

namespace {
int g_captures = 0;          // graphs instantiated
uint64_t g_sel_bytes = 0, g_sel_count = 0;
struct Launch {
    std::string what;
    int grid;
    uint64_t n_known = 0;
    const void *from = nullptr;   // restore: the serialized bytes
    uint32_t n_copy = 0;
};
uint64_t g_spans = 0;        // most bytes that a table's launch copied
bool g_capturing = false;    // the caller's streams
const void *g_copied = nullptr;   // source of the last copy
struct Launches : std::vector<Launch> {
    std::mutex mu;
    void push_back(const Launch &l)
    {
        std::lock_guard<std::mutex> lk(mu);
        std::vector<Launch>::push_back(l);
    }
} g_launches;
// The server's threads meet here: copies of an image to the device, and steps,
// wait (2 s at most) until `wanted` copies are under way at once; the first step
// waits until it is released.
struct Meet {
    std::mutex mu;
    std::condition_variable cv;
    int copies = 0, most = 0, wanted = 0;
    uint64_t bytes = 0;
    bool hold_step = false, in_step = false;
} g_meet;
int handle;                  // streams, events and graphs are its address
}  // namespace

extern "C" {
hipError_t hipMalloc(void **p, size_t n) { *p = calloc(1, (n + 255) & ~size_t(255)); return hipSuccess; }
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void *p) { return hipFree(p); }
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *v, hipDeviceAttribute_t a, int)
{
    *v = a == hipDeviceAttributeMultiprocessorCount ? 256 : 0;
    return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t *e) { *e = (hipEvent_t)&handle; return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { *s = (hipStream_t)&handle; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) { *g = (hipGraph_t)&handle; return hipSuccess; }
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t, hipGraphNode_t *, char *, size_t)
{
    g_captures++;
    *x = (hipGraphExec_t)&handle;
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipSuccess; }
hipError_t hipMemcpy(void *d, const void *s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *d, const void *s, size_t n, hipMemcpyKind k, hipStream_t)
{
    g_copied = s;
    std::unique_lock<std::mutex> lk(g_meet.mu);
    if (g_meet.wanted && k == hipMemcpyHostToDevice && n == g_meet.bytes) {
        g_meet.most = std::max(g_meet.most, ++g_meet.copies);
        g_meet.cv.notify_all();
        g_meet.cv.wait_for(lk, std::chrono::seconds(2), [] { return g_meet.most >= g_meet.wanted; });
        g_meet.copies--;
    }
    lk.unlock();
    return hipMemcpy(d, s, n, k);
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus *c)
{
    CHECK(s);   // the null stream cannot be asked during a capture
    *c = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipMemPrefetchAsync(const void *, size_t, int, hipStream_t) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *s) { *p = const_cast<void *>(s); return hipSuccess; }
}

namespace ckpt {
hipError_t launch_prologue(hipStream_t, const PrologueArgs &a, uint64_t)
{
    uint64_t n = 0;
    for (uint32_t i = 0; i < a.n_copy; i++)
        n += a.copy[i].bytes;
    g_spans = std::max(g_spans, n);
    *a.plan = *a.up_plan;
    return hipSuccess;
}
hipError_t launch_prologue_small(hipStream_t, const PrologueArgs &, const SmallTable &)
{
    g_launches.push_back({"prologue_small", 1});
    return hipSuccess;
}
hipError_t launch_chunks(hipStream_t, int mode, const ChunkArgs &a, int grid, int)
{
    g_launches.push_back({mode == kModeRestore ? "restore" : mode == kModePack ? "pack" : "hash", grid, a.n_known, a.staging});
    return hipSuccess;
}
hipError_t launch_chunks_table(hipStream_t, int, const ChunkArgs &, const SmallTable &, int grid, int)
{
    g_launches.push_back({"chunks_table", grid});
    return hipSuccess;
}
bool table_fits(uint64_t n, uint64_t N, int grid) { return n && n <= kRowTile && N <= (uint64_t)grid * 32; }
hipError_t launch_select(hipStream_t, const SelArgs &a, uint64_t, bool)
{
    if (a.h_plan) {
        a.h_plan->sel_bytes = g_sel_bytes;
        a.h_plan->sel_count = g_sel_count;
    }
    return hipSuccess;
}
hipError_t launch_gather(hipStream_t, const GatherArgs &a, int grid)
{
    g_launches.push_back({a.out_host ? "gather_host" : "gather", grid, 0, nullptr, a.n_copy});
    return hipSuccess;
}
hipError_t launch_pick_u64(hipStream_t, const uint64_t *, const uint64_t *, uint64_t *, uint32_t) { return hipSuccess; }
hipError_t launch_table_split(hipStream_t, const uint64_t *, uint64_t, DevPlan *, uint64_t *, uint64_t *)
{
    g_launches.push_back({"table_split", 1});
    return hipSuccess;
}
hipError_t launch_layout_scan(hipStream_t, DevPlan *, const uint64_t *, uint32_t, uint64_t *, uint64_t *) { return hipSuccess; }
hipError_t launch_chunk_map(hipStream_t, const DevPlan *, const uint64_t *, uint32_t *, int) { return hipSuccess; }
hipError_t launch_rows(hipStream_t, const RowArgs &, int grid, int)
{
    g_launches.push_back({"rows", grid});
    std::unique_lock<std::mutex> lk(g_meet.mu);
    g_meet.in_step = true;
    g_meet.cv.notify_all();
    g_meet.cv.wait_for(lk, std::chrono::seconds(20), [] { return !g_meet.hold_step; });
    g_meet.cv.wait_for(lk, std::chrono::seconds(2), [] { return g_meet.most >= g_meet.wanted; });
    return hipSuccess;
}
// parts of the library that these checks do not enter
std::recursive_mutex &hook_mutex() { static std::recursive_mutex m; return m; }
void hook_forget(ckpt_ctx *) {}
void vmm_release_all(ckpt_ctx *) {}
}  // namespace ckpt

// -------------------------------------------------------------------- checks

namespace {

ckpt_ctx *context(uint32_t flags, uint32_t C = 4096)
{
    ckpt_config cfg;
    memset(&cfg, 0, sizeof(cfg));
    cfg.flags = flags;
    cfg.chunk_bytes = C;
    ckpt_ctx *ctx = nullptr;
    CHECK(ckpt_init(&cfg, &ctx) == CKPT_OK);
    return ctx;
}

// Nothing reads registered memory here.
void log_memory(ckpt_ctx *ctx, uint64_t addr, uint64_t bytes)
{
    ckpt_id id;
    CHECK(ckpt_register(ctx, (void *)addr, bytes, CKPT_DEVICE, &id) == CKPT_OK);
}

ckpt_image *checkpoint(ckpt_ctx *ctx, int mode = CKPT_FULL, const ckpt_image *base = nullptr)
{
    ckpt_image *img = nullptr;
    CHECK(ckpt_checkpoint(ctx, nullptr, mode, base, &img) == CKPT_OK);
    return img;
}

bool has_dense(const ckpt_image *img)
{
    const void *p = nullptr;
    size_t n = 0;
    ckpt_image_meta m;
    CHECK(ckpt_image_info(img, &m) == CKPT_OK);
    const int rc = ckpt_image_view(img, CKPT_SEC_DENSE, &p, &n);
    CHECK(rc == CKPT_OK || (rc == CKPT_E_INVAL && !p && !n));
    CHECK((rc == CKPT_OK) == (m.has_dense != 0));
    return rc == CKPT_OK;
}

// A DENSE view into the context's staging is given only while that memory is there.
void check_dense()
{
    for (uint32_t flags : {CKPT_NO_DRAIN, CKPT_NO_DRAIN | CKPT_GRAPH}) {
        ckpt_ctx *ctx = context(flags);
        log_memory(ctx, 1 << 20, 10000);
        ckpt_image *a = checkpoint(ctx);
        CHECK(has_dense(a));
        ckpt_image *b = checkpoint(ctx);       // the same staging
        CHECK(has_dense(a) && has_dense(b));
        log_memory(ctx, 1 << 30, 64 << 20);    // the staging is replaced by a larger one
        ckpt_image *c = checkpoint(ctx);
        CHECK(!has_dense(a) && !has_dense(b) && has_dense(c));
        ckpt_destroy(ctx);
        CHECK(!has_dense(c));
        for (ckpt_image *x : {a, b, c})
            ckpt_image_free(x);
    }
    // images of a batch point into the first context's staging
    ckpt_ctx *two[2] = {context(CKPT_NO_DRAIN), context(CKPT_NO_DRAIN)};
    log_memory(two[0], 1 << 20, 5000);
    log_memory(two[1], 1 << 30, 7000);
    ckpt_image *img[2];
    CHECK(ckpt_checkpoint_batch(two, 2, nullptr, img) == CKPT_OK);
    ckpt_destroy(two[1]);
    CHECK(has_dense(img[0]) && has_dense(img[1]));
    ckpt_destroy(two[0]);
    CHECK(!has_dense(img[0]) && !has_dense(img[1]));
    // an image that owns its dense copy keeps it
    ckpt_ctx *ctx = context(CKPT_KEEP_DENSE | CKPT_NO_DRAIN);
    log_memory(ctx, 1 << 20, 10000);
    ckpt_image *own = checkpoint(ctx);
    ckpt_destroy(ctx);
    CHECK(has_dense(own));
    for (ckpt_image *x : {img[0], img[1], own})
        ckpt_image_free(x);
}

// One capture, whatever other checkpoints the context takes in between.
void check_graph()
{
    for (uint32_t flags : {0u, (uint32_t)CKPT_NO_DRAIN}) {
        ckpt_ctx *ctx = context(flags | CKPT_GRAPH);
        log_memory(ctx, 1 << 20, 1000000);
        g_captures = 0;
        ckpt_image *base = checkpoint(ctx);
        for (int i = 0; i < 10; i++) {
            for (int k = 0; k <= i % 3; k++)      // an odd and an even number of increments
                ckpt_image_free(checkpoint(ctx, CKPT_INCREMENTAL, base));
            ckpt_image_free(checkpoint(ctx));
            ckpt_image_free(checkpoint(ctx, CKPT_FULL, base));   // with a base: no graph
        }
        CHECK(g_captures == 1);
        ckpt_image_free(base);
        ckpt_destroy(ctx);
    }
    // the first context of a batch, which also takes checkpoints of its own
    ckpt_ctx *two[2] = {context(0), context(0)};
    log_memory(two[0], 1 << 20, 1000000);
    log_memory(two[1], 1 << 30, 500000);
    g_captures = 0;
    for (int i = 0; i < 6; i++) {
        ckpt_image *img[2];
        CHECK(ckpt_checkpoint_batch(two, 2, nullptr, img) == CKPT_OK);
        ckpt_image_free(checkpoint(two[0], CKPT_INCREMENTAL, img[0]));
        ckpt_image_free(img[0]);
        ckpt_image_free(img[1]);
    }
    CHECK(g_captures == 1);
    // many short rows, then as many chunks in few long rows, which are mapped
    // in pieces
    ckpt_ctx *lead = context(CKPT_NO_DRAIN, 16), *rows = context(0, 16), *lengths = context(0, 16);
    for (uint64_t k = 0; k < 10000; k++)
        log_memory(rows, (1 << 20) + 512 * k, 512);
    for (uint64_t k = 0; k < 70; k++)
        log_memory(lengths, (1 << 30) + 65664 * k, 65664);   // 4104 chunks
    g_captures = 0;
    for (int i = 0; i < 4; i++)
        for (ckpt_ctx *x : {rows, lengths}) {
            ckpt_ctx *pair[2] = {lead, x};
            ckpt_image *img[2];
            CHECK(ckpt_checkpoint_batch(pair, 2, nullptr, img) == CKPT_OK);
            ckpt_image_free(img[0]);
            ckpt_image_free(img[1]);
        }
    CHECK(g_captures == 1);
    for (ckpt_ctx *x : {two[0], two[1], lead, rows, lengths})
        ckpt_destroy(x);
}

bool launched(const char *what)
{
    for (const Launch &l : g_launches)
        if (l.what == what)
            return true;
    return false;
}

// Outside a capture the host's table and counts go with the launches; a
// captured pass takes both from the log when it is replayed.
void check_capture()
{
    static uint8_t out[1 << 22] __attribute__((aligned(256)));
    for (uint64_t n : {5, 64, 65}) {
        ckpt_ctx *ctx = context(CKPT_STREAM_ORDERED);
        for (uint64_t k = 0; k < n; k++)
            log_memory(ctx, (1 << 30) + 65536 * k, 10000 + k);
        for (int mode : {CKPT_FULL, CKPT_INCREMENTAL})
            for (bool capturing : {false, true}) {
                g_capturing = capturing;
                g_launches.clear();
                g_copied = nullptr;
                uint64_t N = 0;
                CHECK(ckpt_checkpoint_noalloc(ctx, (void *)&handle, mode, (uint32_t *)out, out, sizeof(out),
                                              (uint32_t *)out, out, 4096, &N, nullptr) == CKPT_OK);
                CHECK(N == 3 * n);
                if (capturing || n > 64) {
                    CHECK(launched("table_split") && !launched("chunks_table") && !launched("prologue_small"));
                    CHECK(g_copied == ctx->live.data());
                    CHECK(g_launches.back().n_known == (capturing ? 0 : N));
                } else {
                    CHECK(launched("chunks_table") && !g_copied);
                }
            }
        g_capturing = false;
        CHECK(ckpt_checkpoint_noalloc(ctx, nullptr, CKPT_FULL, nullptr, out, sizeof(out), (uint32_t *)out, out, 4096,
                                      nullptr, nullptr) == CKPT_OK);
        ckpt_destroy(ctx);
    }
}

// What a drain of n allocations of `bytes` each, of which `ser` bytes are
// serialized, launches, and then a refill of the image.
struct Route {
    bool drain_direct, refill_direct;
    int refill_grid;
};
Route route(uint32_t C, uint64_t n, uint64_t bytes, uint64_t ser)
{
    ckpt_ctx *ctx = context(0, C);
    std::vector<void *> dst(n);
    for (uint64_t k = 0; k < n; k++) {
        dst[k] = (void *)((uint64_t(1) << 32) + (bytes + 4096) / 4096 * 4096 * k);
        log_memory(ctx, (uint64_t)dst[k], bytes);
    }
    g_sel_bytes = ser;
    Route r{};
    g_launches.clear();
    ckpt_image *img = checkpoint(ctx);
    CHECK(img->ser_bytes == ser);
    r.drain_direct = launched("gather_host");
    CHECK(r.drain_direct != launched("gather") || !ser);
    g_launches.clear();
    CHECK(ckpt_restore(ctx, nullptr, img, nullptr, dst.data(), nullptr, n, nullptr) == CKPT_OK);
    g_sel_bytes = 0;
    CHECK(g_launches.size() && g_launches[0].what == "restore");
    r.refill_grid = g_launches[0].grid;
    r.refill_direct = g_launches[0].from == img->data.p;
    ckpt_image_free(img);
    ckpt_destroy(ctx);
    return r;
}

// Kernels reach over the link for a MiB at most (others wait meanwhile); the
// rest goes through staging, and refills take the whole chip.
void check_link()
{
    const uint64_t M = 1 << 20;
    for (uint32_t C : {16, 4096, 65536}) {
        for (uint64_t ser : {uint64_t(16), M}) {
            const Route r = route(C, 1, M, ser);
            CHECK(r.drain_direct && r.refill_direct && r.refill_grid == 256);
        }
        for (uint64_t bytes : {M + 16, 9 * M, 16 * M, 240 * M}) {
            if (bytes / C > 4 * M)
                continue;
            Route r = route(C, 1, bytes, bytes);
            CHECK(!r.drain_direct && !r.refill_direct && r.refill_grid == 256);
            r = route(C, 1, bytes, M / 2);
            CHECK(r.drain_direct && r.refill_direct && r.refill_grid == 256);
        }
    }
    // more chunks than a segment has, and few bytes
    CHECK(route(65536, 5000, 100, 5000 * 112).drain_direct);
    // an increment's ids and bytes, and its refill
    ckpt_ctx *ctx = context(0, 16);
    log_memory(ctx, 1 << 20, 64 * M);
    g_sel_bytes = 64 * M;
    ckpt_image *base = checkpoint(ctx);
    for (uint64_t ser : {uint64_t(0), M, M + 16}) {
        for (uint64_t count : {M / 8, M / 8 + 1}) {
            g_sel_bytes = ser;
            g_sel_count = count;
            g_launches.clear();
            ckpt_image *delta = checkpoint(ctx, CKPT_INCREMENTAL, base);
            CHECK(launched("gather_host") == (ser == M) && launched("gather") == (ser > M));
            if (ser)
                CHECK(g_launches.back().n_copy == (count == M / 8 ? 1 : 0));
            for (uint64_t i = 0; i < count; i++)   // no kernel has written the ids
                ((uint64_t *)delta->ids_buf.p)[i] = i;
            void *dst = (void *)(1 << 20);
            g_launches.clear();
            CHECK(ckpt_restore(ctx, nullptr, base, delta, &dst, nullptr, 1, nullptr) == CKPT_OK);
            CHECK(g_launches.size() == 2 && g_launches[0].from != base->data.p && g_launches[1].grid == 256);
            CHECK((g_launches[1].from == delta->data.p) == (ser <= M));
            ckpt_image_free(delta);
        }
    }
    g_sel_bytes = g_sel_count = 0;
    CHECK(g_spans <= M);
    ckpt_image_free(base);
    ckpt_destroy(ctx);
}

uint64_t submit(ckpt_server *sv, int op, void *ptr, uint64_t size, ckpt_image *img)
{
    ckpt_request q;
    memset(&q, 0, sizeof(q));
    q.op = op;
    q.n = 1;
    q.ptrs = &ptr;
    q.sizes = &size;
    q.image = img;
    uint64_t t = 0;
    CHECK(ckpt_server_submit(sv, &q, &t) == CKPT_OK);
    return t;
}

// Restores are copied to the device by every free worker, also while a
// checkpoint is being packed; a checkpoint's chunks are gathered to the device
// and copied from there.
void check_server()
{
    const uint64_t bytes = 8 << 20;
    ckpt_ctx *ctx = context(0);
    log_memory(ctx, 1 << 30, bytes);
    g_sel_bytes = g_meet.bytes = bytes;
    ckpt_image *img = checkpoint(ctx);
    ckpt_server_config cfg;
    memset(&cfg, 0, sizeof(cfg));
    cfg.chunk_bytes = 4096;
    cfg.staging_budget = 256 << 20;
    cfg.aux_threads = 4;
    cfg.step_bytes = 1 << 20;   // several steps: requests join between them
    ckpt_server *sv = nullptr;
    CHECK(ckpt_server_create(&cfg, &sv) == CKPT_OK);
    g_launches.clear();
    g_meet.hold_step = true;
    std::vector<uint64_t> tickets{submit(sv, CKPT_REQ_CHECKPOINT, (void *)(1 << 30), bytes, nullptr)};
    {
        std::unique_lock<std::mutex> lk(g_meet.mu);
        CHECK(g_meet.cv.wait_for(lk, std::chrono::seconds(20), [] { return g_meet.in_step; }));
        g_meet.wanted = 3;
    }
    for (int i = 0; i < 3; i++)
        tickets.push_back(submit(sv, CKPT_REQ_RESTORE, (void *)(1 << 30), bytes, img));
    {
        std::lock_guard<std::mutex> lk(g_meet.mu);
        g_meet.hold_step = false;
        g_meet.cv.notify_all();
    }
    for (uint64_t t : tickets) {
        ckpt_result r;
        CHECK(ckpt_server_wait(sv, t, &r) == CKPT_OK && r.status == CKPT_OK);
        if (r.image)
            ckpt_image_free(r.image);
    }
    g_sel_bytes = 0;
    CHECK(g_meet.most == 3);
    CHECK(launched("gather") && !launched("gather_host"));
    ckpt_server_destroy(sv);
    ckpt_image_free(img);
    ckpt_destroy(ctx);
}

}  // namespace

int main(int argc, char **argv)
{
    const std::string what = argc > 1 ? argv[1] : "";
    if (what == "dense")
        check_dense();
    else if (what == "graph")
        check_graph();
    else if (what == "server")
        check_server();
    else if (what == "link")
        check_link();
    else if (what == "capture")
        check_capture();
    else
        return 2;
    printf("all checks held\n");
    return 0;
}
