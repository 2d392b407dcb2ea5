// The two launches of a step whose merges are a launch of their own, as the host code enqueues them: two threads on one context and one
// stream, calls that are recorded into a graph.  Built and run by tests/test_launch_pairs_host.py.
#include <cstdio>
#include <thread>
#include <vector>

#include "hip_host.h"
#include "taper_internal.h"

#define CHECK(cond)                                                                                     \
    do {                                                                                                \
        if (!(cond)) {                                                                                  \
            std::fprintf(stderr, "%s:%d: %s failed (%s)\n", __FILE__, __LINE__, #cond, taper_last_error()); \
            return 1;                                                                                   \
        }                                                                                               \
    } while (0)

// What the stream holds: an entry per launch, the caller's query pointer in it.
struct Launch {
    const void* q;
    bool merge;
};
static std::vector<Launch> stream(1 << 16);
static std::atomic<size_t> n_launches{0};
static taper::StepArgs seen;  // the last call's, while there is one thread
static bool threads = false;
namespace taper {
hipError_t launch_decode(const StepArgs& a, hipStream_t) {
    stream[n_launches++] = {a.q, false};
    for (int i = 0; i < 20; ++i) std::this_thread::yield();  // (another thread's chance)
    if (a.merge_after) stream[n_launches++] = {a.q, true};
    if (!threads) seen = a;
    return hipSuccess;
}
}  // namespace taper

static taper_plan* build(taper_ctx* ctx, int n_tokens) {  // one sequence alone on one kv head: many pieces
    std::vector<int32_t> bt((n_tokens + 15) / 16);
    for (size_t i = 0; i < bt.size(); ++i) bt[i] = (int32_t)i;
    const int32_t zero = 0, len = n_tokens;
    taper_plan* p = nullptr;
    if (taper_plan_build(ctx, 1, bt.data(), (int)bt.size(), &zero, &zero, &len, (int64_t)bt.size(), nullptr, nullptr, &p) != TAPER_OK) return nullptr;
    return p;
}

int main() {
    taper_attn_config cfg = {8, 1, 128, 16, 0.0884f, 0, 0};
    taper_ctx* ctx = nullptr;
    CHECK(taper_create(&cfg, &ctx) == TAPER_OK);
    taper_plan *a = build(ctx, 16000), *b = build(ctx, 15000);
    CHECK(a && b);
    taper_plan_view va, vb;
    CHECK(taper_plan_export(a, &va) == TAPER_OK && taper_plan_export(b, &vb) == TAPER_OK);
    CHECK(va.merge_launch == 1 && vb.merge_launch == 1 && va.workspace_id == vb.workspace_id);
    char tensors[2][4];
    int step = 0;

    // calls that are recorded use other rows of the workspace than eager ones: both whole, and apart
    auto rows_of = [&](taper_plan* p, bool recorded) {
        hip_host::capturing = recorded;
        step = taper_decode_step_attention(ctx, p, tensors[0], tensors[1], tensors[0], nullptr, nullptr);
        hip_host::capturing = 0;
        return seen;
    };
    const taper::StepArgs sets[2] = {rows_of(a, false), rows_of(a, true)};
    CHECK(step == TAPER_OK && sets[0].merge_after && sets[0].counters == sets[1].counters);  // (counters matter inside one launch only)
    struct Range {
        char *first, *end;
    } r[4];
    for (int i = 0; i < 2; ++i) {
        r[2 * i] = {(char*)sets[i].ws_ml, (char*)sets[i].ws_ml + va.workspace_rows * 16};
        r[2 * i + 1] = {(char*)sets[i].ws_o, (char*)sets[i].ws_o + va.workspace_rows * 128 * 2};
    }
    for (int i = 0; i < 4; ++i) {
        CHECK(((uintptr_t)r[i].first & 15) == 0 && hip_host::inside_one_allocation(sets[0].counters, r[i].end));
        for (int k = 0; k < i; ++k) CHECK(r[i].end <= r[k].first || r[k].end <= r[i].first);
    }

    // two threads: launches come in pairs
    threads = true;
    n_launches = 0;
    auto caller = [&](taper_plan* p, char* q) {
        for (int i = 0; i < 4000; ++i) (void)taper_decode_step_attention(ctx, p, q, q, q, nullptr, nullptr);
    };
    std::thread t0(caller, a, tensors[0]), t1(caller, b, tensors[1]);
    t0.join();
    t1.join();
    CHECK(n_launches == 16000);
    size_t changes = 0;
    for (size_t i = 0; i < n_launches; i += 2) {
        if (stream[i].merge || !stream[i + 1].merge || stream[i].q != stream[i + 1].q) {
            std::fprintf(stderr, "launch %zu: attention and merge of different calls\n", i);
            return 1;
        }
        changes += i > 0 && stream[i].q != stream[i - 2].q;
    }
    std::printf("calls taken in turns %zu times\n", changes);

    taper_plan_free(a);
    taper_plan_free(b);
    taper_destroy(ctx);
    CHECK(hip_host::live_allocations() == 0);
    std::puts("ok");
    return 0;
}
