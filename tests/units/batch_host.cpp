// The host side of the batch calls (csrc/batch.cpp) and of the server (csrc/serve.cpp) over a runtime that does no GPU work: it logs the calls and
// fails the one it is told to.  argv: a scenario; prints the log, one call a line.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <string>

#include "../../paper_1305_4376_amd/csrc/batch_plan.h"
#include "../../paper_1305_4376_amd/csrc/internal.h"

namespace {

std::string g_fail;                 // the runtime call that fails
hipError_t g_last = hipSuccess;     // the error the next hipGetLastError reports
hipStream_t g_capturing = nullptr;  // the stream under capture

void log(const char *what) { printf("%s\n", what); }

hipError_t result(const char *call) {
    if (g_fail != call) return hipSuccess;
    return g_last = hipErrorUnknown;
}

// A launcher's end, as the library's are: any error left behind fails it.
hipError_t launched(const char *what, hipStream_t s) {
    log((std::string(s && s == g_capturing ? "capture " : "launch ") + what).c_str());
    return hipGetLastError();
}

char g_objects[64];
int g_next = 0;
template <class T>
hipError_t make(T *out) {
    *out = reinterpret_cast<T>(&g_objects[g_next++ % 64]);
    return hipSuccess;
}

}  // namespace

extern "C" {
hipError_t hipGetDevice(int *d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceCount(int *n) { *n = 1; return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() { const hipError_t e = g_last; g_last = hipSuccess; return e; }
hipError_t hipMalloc(void **p, size_t n) { *p = malloc(n); return hipSuccess; }
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipHostMalloc(void **p, size_t n, unsigned) { *p = malloc(n); return hipSuccess; }
hipError_t hipHostFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemset(void *p, int v, size_t n) { memset(p, v, n); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t *s, unsigned) { return make(s); }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipMemcpyAsync(void *to, const void *from, size_t n, hipMemcpyKind, hipStream_t) { memcpy(to, from, n); return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) { return make(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode) {
    if (result("begin") != hipSuccess) return hipErrorUnknown;
    g_capturing = s;
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *g) {
    g_capturing = nullptr;
    if (result("end") != hipSuccess) return hipErrorUnknown;
    return make(g);
}
hipError_t hipGraphInstantiate(hipGraphExec_t *x, hipGraph_t, hipGraphNode_t *, char *, size_t) {
    if (result("instantiate") != hipSuccess) return hipErrorUnknown;
    log("instantiate");
    return make(x);
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { log("drop graph"); return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { log("launch graph"); return hipSuccess; }
}

namespace tdes {
int device_info(DeviceInfo *info) {
    *info = DeviceInfo{256, 0};
    return TDES_OK;
}
hipError_t launch_auto(const uint32_t *, const uint8_t *, uint8_t *, uint64_t, hipStream_t s) { return launched("message", s); }
hipError_t launch_plan(const PlanMessage *, uint32_t, uint32_t, PlanHeader *, Slot *, uint32_t, uint32_t, hipStream_t s) {
    return launched("plan", s);
}
hipError_t launch_fill_tiles(const FillTile *, uint32_t, uint8_t *, hipStream_t s) { return launched("fill", s); }
hipError_t launch_batch(const uint32_t *, const PlanHeader *, const Slot *, uint32_t *, uint8_t *, uint32_t, uint32_t,
                        uint32_t, bool, hipStream_t s) {
    return launched("waves", s);
}
hipError_t launch_batch_team(const uint32_t *, const PlanHeader *, const Slot *, uint8_t *, uint32_t, hipStream_t s) {
    return launched("teams", s);
}
}  // namespace tdes

namespace {

alignas(16) uint8_t g_table[TDES_SCHED_BYTES], g_base[2][64];

void batch(tdes_ctx *c, uint64_t n_blocks, uint8_t *base, uint32_t flags = 0) {
    tdes_job job{};
    job.out_off = 8 * n_blocks;
    job.n_blocks = n_blocks;
    printf("batch %d\n", tdes_ecb_batch(c, &job, 1, g_table, 1, base, flags, nullptr));
}

// A server with one step in flight: two requests of n blocks, one after the other.
int serve(uint64_t n) {
    tdes_serve_config cfg{};
    cfg.budget_bytes = 16 * n + 4096;
    cfg.max_inflight = 1;
    cfg.max_step_jobs = 8;
    cfg.max_step_blocks = n;
    tdes_server *s = nullptr;
    if (tdes_server_create(&s, &cfg, g_table, 1) != TDES_OK) return 2;
    for (int i = 0; i < 2; i++) {
        tdes_request r{};
        r.n_blocks = n;
        const int rc = tdes_server_submit(s, &r, nullptr), idle = tdes_server_wait_idle(s, 30);
        printf("served %d %d\n", rc, idle);
    }
    return tdes_server_destroy(s);
}

void replay(tdes_ctx *c) { printf("replay %d\n", tdes_ecb_batch_replay(c, 0, nullptr)); }

}  // namespace

int main(int argc, char **argv) {
    setvbuf(stdout, nullptr, _IOLBF, 0);
    const std::string what = argc > 1 ? argv[1] : "";
    const uint64_t n = argc > 2 ? strtoull(argv[2], nullptr, 10) : 100;
    if (what == "serve") return serve(n);
    tdes_ctx *c = nullptr;
    if (tdes_ctx_create(&c, 0) != TDES_OK) return 2;
    if (what == "ordinary") {
        batch(c, n, g_base[0]);
        replay(c);
        batch(c, n, g_base[0]);
        batch(c, n, g_base[1]);
        replay(c);
        batch(c, n, g_base[0], TDES_BATCH_NO_GRAPH);
    } else {  // the capture's call of this name fails, and later works again
        g_fail = what;
        batch(c, n, g_base[0]);
        batch(c, n, g_base[0]);
        replay(c);
        g_fail = "";
        replay(c);
    }
    tdes_ctx_destroy(c);
    return 0;
}
