// The start records of plans: what each wave's first loads are made from, against the items and the block table.  Built and run by
// tests/test_start_records_host.py.
#include <cstdio>
#include <random>

#include "taper_plan.h"

using namespace taper;

static int page_of(const HostPlan& p, const taper_work_item& it, int i) {  // the item's i-th page, past its end the last one
    const int n = (it.n_tokens + 15) / 16;
    return p.block_table[(size_t)it.seq0 * p.bt_stride + it.page0 + (i < n ? i : n - 1)];
}

int main() {
    std::mt19937 rng(7);
    auto pick = [&](int lo, int hi) { return lo + (int)(rng() % (unsigned)(hi - lo + 1)); };
    int checked[4] = {0, 0, 0, 0};  // shared, private, solo, shares of more than one item
    for (int round = 0; round < 400; ++round) {
        const int shapes[5][3] = {{64, 8, 128}, {8, 1, 128}, {6, 2, 128}, {32, 8, 64}, {16, 1, 64}};
        const int* s = shapes[round % 5];
        const taper_attn_config cfg = {s[0], s[1], s[2], 16, 0.1f, -1, 0};
        std::vector<int32_t> group, prefix, suffix;
        for (int g = 0, n = pick(1, 12); g < n; ++g) {
            const int top = 1 << pick(4, 12), pl = pick(0, 3) ? pick(1, top) : 0;
            for (int b = 0, w = pick(0, 2) ? 1 : pick(2, 30); b < w; ++b) {
                group.push_back(g);
                prefix.push_back(pl);
                suffix.push_back(pl && pick(0, 3) == 0 ? 0 : pick(1, 1 << pick(3, 11)));
            }
        }
        const int n = (int)group.size();
        int stride = 1;
        for (int i = 0; i < n; ++i) stride = std::max(stride, (prefix[i] + 15) / 16 + (suffix[i] + 15) / 16);
        std::vector<int32_t> bt((size_t)n * stride, -1);
        for (int i = 0; i < n; ++i) {
            const int shared = (prefix[i] + 15) / 16, all = shared + (suffix[i] + 15) / 16;
            for (int j = 0; j < all; ++j)
                bt[(size_t)i * stride + j] = j < shared && i > 0 && group[i] == group[i - 1] ? bt[(size_t)(i - 1) * stride + j] : pick(0, 99999);
        }
        taper_plan_options o = {};
        o.share_prefix = 1;
        o.target_workgroups = round % 3 ? 512 : s[1] * pick(1, 9);
        o.small_step_grid = round % 2;
        HostPlan p;
        std::string err;
        if (build_host_plan(cfg, n, bt.data(), stride, group.data(), prefix.data(), suffix.data(), 100000, &o, &p, &err) != TAPER_OK) {
            std::printf("round %d: %s\n", round, err.c_str());
            return 1;
        }
        const int n_parts = p.n_parts_shared + p.n_parts_private;
        if (p.starts.size() * sizeof(StartWords) != (size_t)n_parts * p.start_bytes) return 2;
        for (int q = 0; q < n_parts; ++q) {
            const int first = p.part_start[q], end = p.part_start[q + 1], n_solo = p.part_turn[q] >> kPartSoloShift;
            if (first == end) return 3;
            checked[3] += end - first > 1;
            for (int w = 0; w < 4; ++w) {
                const ShareStart& r = *(const ShareStart*)((const char*)p.starts.data() + (size_t)q * p.start_bytes);
                const bool solo = w < n_solo;
                const taper_work_item& it = p.items[solo ? first + w : first];
                const taper_work_item& has = r.item[p.start_bytes == kStartBytesFour ? w : 0];
                if (p.start_bytes == kStartBytesOne && n_solo > 1) return 6;
                bool ok = r.first == first && r.end == end && r.n_solo == n_solo && r.turn == (p.part_turn[q] & ((1 << kPartSoloShift) - 1)) &&
                          (r.turn & kPartTurnMask) < s[1] && has.seq0 == it.seq0 && has.n_tokens == it.n_tokens && has.page0 == it.page0 &&
                          has.kind == it.kind && has.part_base == it.part_base && has.merge0 == it.merge0 && has.n_branch == it.n_branch;
                for (int block = 0; block < 2 && it.kind != 0; ++block)  // a wave's first two blocks, two pages each
                    for (int half = 0; half < 2; ++half) ok &= r.page[w][2 * block + half] == page_of(p, it, 2 * (solo ? block : w + 4 * block) + half);
                for (int i = 0; i < 4 && it.kind == 0; ++i) {  // the first four blocks: of two pages, which every wave stages a part of, or of four, a page a wave
                    if (s[2] == 128) ok &= r.page[w][i] == page_of(p, it, i) && r.more[i] == page_of(p, it, 4 + i);
                    else ok &= r.page[w][i] == page_of(p, it, 4 * i + w);
                }
                if (!ok) {
                    std::printf("round %d share %d wave %d\n", round, q, w);
                    return 4;
                }
                checked[solo ? 2 : it.kind != 0]++;
            }
        }
    }
    std::printf("shared %d private %d solo %d, shares of several items %d\n", checked[0], checked[1], checked[2], checked[3]);
    return checked[0] && checked[1] && checked[2] && checked[3] ? 0 : 5;
}
