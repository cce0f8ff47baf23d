// Steps that are queued without their routing, on a machine without a GPU: this file is the library (its source is included
// below) with launches that only count, and fail where a check wants one to.  Built for the host alone and run by
// tests/test_queued_steps.py; prints "ok" and exits 0 when nothing was found.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

static int g_launches = 0, g_fail_at = -1;               // launches so far; the one that fails
static hipError_t launch_result() { return g_launches - 1 == g_fail_at ? hipErrorLaunchFailure : hipSuccess; }

#undef hipLaunchKernelGGL
#define hipLaunchKernelGGL(...) (void)++g_launches
#undef hipExtLaunchKernelGGL
#define hipExtLaunchKernelGGL(...) (void)++g_launches
#define hipGetLastError() launch_result()
#define hipStreamSynchronize(s) ((void)(s), hipSuccess)
#define hipFuncSetAttribute(...) hipSuccess
#define hipEventCreate(e) (*(e) = nullptr, hipSuccess)
#define hipEventSynchronize(e) hipSuccess
#define hipEventRecord(e, s) hipSuccess
#define hipEventElapsedTime(ms, a, b) (*(ms) = 1.f, hipSuccess)
#define hipMemcpy(d, s, n, k) (memcpy(d, s, n), hipSuccess)
#include "../../paper_2312_17238_amd/csrc/moe_offload.hip"

// no device code: nothing to register
extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *handle; return &handle; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *, char *, const char *, unsigned, uint3 *, uint3 *, dim3 *, dim3 *, int *) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
const char __hip_fatbin[8] = {0};
}

#define CHECK(cond)                                                                         \
    do {                                                                                    \
        if (!(cond)) {                                                                      \
            std::fprintf(stderr, "%s:%d: check failed: %s (last error: %s)\n", __FILE__, __LINE__, #cond, moe_last_error()); \
            std::exit(1);                                                                   \
        }                                                                                   \
    } while (0)

// A context and one layer with all experts resident.  Its memory is never touched by anything that runs here, the log of
// selections excepted, which the checks write in the kernels' place.
struct Layer {
    moe_ctx *ctx = nullptr;
    moe_layer *layer = nullptr;
    std::vector<uint8_t> host;
    std::vector<int32_t> log, log_dev;
    std::vector<uint16_t> x;

    Layer(int H, int F, int E, int K, int bits, int group, int batch)
    {
        const uint64_t blob = moe_expert_blob_bytes(H, F, bits, group);
        moe_ctx_config_t cc{0, batch, H, F, K, MOE_CTX_HOST_ONLY, blob};
        CHECK(moe_ctx_create(&cc, nullptr, 0, nullptr, nullptr, &ctx) == MOE_OK);
        host.resize(blob * E + 64);
        moe_layer_config_t lc{H, F, E, K, bits, group, E, 0, 1e-5f, 1, 0, 0};
        std::vector<float> gate((size_t)E * H, 0.f);
        CHECK(moe_layer_create(ctx, &lc, gate.data(), nullptr, nullptr, host.data() + (64 - (uintptr_t)host.data() % 64) % 64, &layer) == MOE_OK);
        for (int e = 0; e < E; ++e)
            for (int m = 0; m < 3; ++m) {
                const size_t rows = m == 2 ? H : F, cols = m == 2 ? F : H;
                std::vector<uint8_t> q(rows * cols, 1);
                std::vector<uint16_t> s(rows * cols / group, 0x3c00), z(rows * cols / group, 0);
                CHECK(moe_layer_load_expert(layer, e, m, q.data(), s.data(), z.data()) == MOE_OK);
            }
        log.resize((size_t)moe_ctx::ROUTE_LOG * MOE_MAX_TOPK);
        log_dev = log;
        x.resize((size_t)batch * H);
        ctx->route_log = log.data();
        ctx->route_log_dev = log_dev.data();
        ctx->n_cu = 256;
        ctx->ypart_extra_floats = plan_scratch(&cc).ypart_extra_floats;
        ctx->host_only = false;          // from here on it steps
    }
    ~Layer()
    {
        ctx->host_only = true;
        CHECK(moe_layer_destroy(layer) == MOE_OK && moe_ctx_destroy(ctx) == MOE_OK);
    }
    int32_t step(int batch) { g_launches = 0; return moe_layer_step(layer, nullptr, x.data(), batch, x.data(), nullptr, nullptr); }
    void selected(uint32_t mask) { log_dev[(size_t)ctx->pending.back().slot * MOE_MAX_TOPK] = (int32_t)mask; }
    moe_stats_t stats()
    {
        moe_stats_t s;
        CHECK(moe_layer_stats(layer, &s) == MOE_OK);
        return s;
    }
};

// A step one of whose launches fails leaves nothing behind that the bookkeeping would read from a log word nobody wrote.
static void failed_launches(int bits, int group, int batch, int min_batch, BatchPlan::Kind kind)
{
    Layer l(256, 512, 8, 2, bits, group, batch);
    CHECK(moe_ctx_set_option(l.ctx, "mfma_min_batch", min_batch) == MOE_OK);
    CHECK(plan_batch(l.layer, batch).kind == kind);
    CHECK(l.step(batch) == MOE_OK && l.ctx->pending.size() == 1);
    l.selected(0x15);
    const int launches = g_launches;
    moe_stats_t s = l.stats();
    CHECK(launches >= 4 && s.steps == 1 && s.steps_device_routed == 1 && s.needed == 3 && s.hits == 3);
    for (g_fail_at = 0; g_fail_at < launches; ++g_fail_at) {
        l.log_dev.assign(l.log_dev.size(), 0x7fffffff);
        CHECK(l.step(batch) != MOE_OK && g_launches == g_fail_at + 1);
        CHECK(l.ctx->pending.empty());
        s = l.stats();
        CHECK(s.steps == 1 && s.steps_device_routed == 1 && s.needed == 3);
    }
    g_fail_at = -1;
    CHECK(l.step(batch) == MOE_OK);
    l.selected(0x80);
    s = l.stats();
    CHECK(s.steps == 2 && s.steps_device_routed == 2 && s.needed == 4 && s.hits == 4);
}

// Algorithmic bytes: the experts that a step turned out to need, once each.
static void profiled_bytes(int bits, int group, int batch, int min_batch)
{
    Layer l(256, 512, 8, 2, bits, group, batch);
    CHECK(moe_ctx_set_option(l.ctx, "mfma_min_batch", min_batch) == MOE_OK);
    CHECK(l.step(batch) == MOE_OK);              // not timed
    l.selected(0xff);
    CHECK(moe_ctx_profile_enable(l.ctx, 1) == MOE_OK);
    const uint32_t masks[3] = {0x01, 0x90, 0xff};
    for (uint32_t m : masks) { CHECK(l.step(batch) == MOE_OK); l.selected(m); }
    const MatLayout &m13 = l.layer->lay.m13, &m2 = l.layer->lay.m2;
    moe_profile_t p;
    CHECK(moe_ctx_profile_read(l.ctx, &p) == MOE_OK);
    CHECK(p.w13.launches == 3 && p.w13.bytes == 11ull * 2 * 512 * m13.row_stride);
    CHECK(p.w2.launches == 3 && p.w2.bytes == 11ull * 256 * m2.row_stride);
    CHECK(l.step(batch) == MOE_OK);
    l.selected(0x03);
    CHECK(moe_ctx_profile_enable(l.ctx, 1) == MOE_OK);       // clears
    CHECK(moe_ctx_profile_read(l.ctx, &p) == MOE_OK && p.w13.bytes == 0 && p.w2.bytes == 0);
    const moe_stats_t s = l.stats();
    CHECK(s.steps == 5 && s.needed == 8 + 11 + 2);
}

int main()
{
    failed_launches(3, 64, 4, 1000, BatchPlan::GEMV);
    failed_launches(4, 64, 8, 3, BatchPlan::STREAM);
    failed_launches(3, 64, 40, 3, BatchPlan::TILE);
    failed_launches(3, 64, 200, 3, BatchPlan::TILE);          // ... with the sorted list
    profiled_bytes(3, 64, 4, 1000);
    profiled_bytes(4, 64, 8, 3);
    profiled_bytes(3, 64, 40, 3);
    std::printf("ok\n");
    return 0;
}
