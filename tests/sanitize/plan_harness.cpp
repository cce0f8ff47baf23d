// What the library plans for a batch, on a machine without a GPU: built and run by tests/test_plans.py with the layer, the batch and the tokens of a
// block as arguments, and the form if not the tile kernels'.  Prints how many parts w2 has with an even routing and with every token at the same experts, the calls of erfc that the plan
// took and the tokens of a block of w2; four zeros where other kernels run the step.
#include <hip/hip_runtime.h>
#include <cmath>
static int g_erfc = 0;
namespace std { static double counted_erfc(double x) { ++g_erfc; return (erfc)(x); } }
#define erfc counted_erfc
#define main queued_steps_main
#include "queued_steps_harness.cpp"
#undef main

int main(int argc, char **argv)
{
    CHECK(argc == 10 || argc == 11);
    int v[10] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 6};
    for (int i = 1; i < argc; ++i) v[i - 1] = atoi(argv[i]);
    const int bits = v[0], group = v[1], scale_group = v[2], H = v[3], F = v[4], E = v[5], K = v[6], batch = v[7];
    const BlobLayout b = blob_layout(H, F, bits, group, scale_group);
    CHECK(b.ok);
    moe_ctx *ctx = nullptr;
    moe_layer *layer = nullptr;
    moe_ctx_config_t cc{0, batch, H, F, K, MOE_CTX_HOST_ONLY, b.total};
    CHECK(moe_ctx_create(&cc, nullptr, 0, nullptr, nullptr, &ctx) == MOE_OK);
    moe_layer_config_t lc{H, F, E, K, bits, group, E, 0, 1e-5f, 1, 0, scale_group};
    std::vector<float> gate((size_t)E * H, 0.f);
    std::vector<uint8_t> host(b.total * E + 64);
    CHECK(moe_layer_create(ctx, &lc, gate.data(), nullptr, nullptr, host.data() + (64 - (uintptr_t)host.data() % 64) % 64, &layer) == MOE_OK);
    layer->scale_top.store(0x3c000000);                  // 2^-7: what the 2-bit tile kernels ask of a layer's scales
    layer->scale_row_low.store(0x3c000000);
    ctx->n_cu = 256;
    ctx->ypart_extra_floats = plan_scratch(&cc).ypart_extra_floats;
    ctx->mfma_form = v[9];
    ctx->tile_tokens = v[8];
    g_erfc = 0;
    const BatchPlan p = plan_batch(layer, batch);
    if (p.kind != BatchPlan::TILE) { CHECK(v[9] != 6); std::puts("0 0 0 0"); return 0; }
    const int sets = (F / 64 + 3) / 4, blocks = K * tile_blocks(b, batch, p.mode2);
    int32_t even, crowded, units;
    te_split(sets, p.parts, even, units);
    te_split(sets, blocks < p.few_below ? p.few[blocks - 1] : p.parts, crowded, units);
    std::printf("%d %d %d %d\n", even, crowded, g_erfc, p.mode2 == TE_BIG ? 192 : p.mode2);
    CHECK(moe_layer_destroy(layer) == MOE_OK && moe_ctx_destroy(ctx) == MOE_OK);
    return 0;
}
