// Host-side index resolution for one decode step (see taper_plan.h).
//
// Which KV each query row reads follows the visibility rule (paper §3.1): the
// request's shared prefix, then the sequence's own private tokens.  The shared
// prefix of a request with several admitted branches becomes "shared" work
// (read once, multiplied against all branches' query rows); everything else is
// "private" work (one sequence's rows).
#include "taper_plan.h"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <functional>
#include <cstring>

namespace taper {

static std::string fmt(const char* f, long long a = 0, long long b = 0, long long c = 0) {
    char buf[256];
    std::snprintf(buf, sizeof buf, f, a, b, c);
    return buf;
}

int validate_config(const taper_attn_config& cfg, std::string* err) {
    if (cfg.n_q_heads < 1 || cfg.n_kv_heads < 1 || cfg.n_q_heads % cfg.n_kv_heads != 0) {
        *err = "n_q_heads must be a positive multiple of n_kv_heads";
        return TAPER_EINVAL;
    }
    int g = cfg.n_q_heads / cfg.n_kv_heads;
    if (g > 16) {
        *err = "at most 16 query heads per KV head are supported";
        return TAPER_EINVAL;
    }
    if (cfg.head_dim != 64 && cfg.head_dim != 128) {
        *err = "head_dim must be 64 or 128";
        return TAPER_EINVAL;
    }
    if (cfg.page_size != 16) {
        *err = "page_size must be 16";
        return TAPER_EINVAL;
    }
    if (!(cfg.scale > 0.0f) || !(cfg.scale < 1e30f)) {
        *err = "scale must be positive and finite";
        return TAPER_EINVAL;
    }
    if (cfg.partial_format != TAPER_PARTIAL_F16_SCALED && cfg.partial_format != TAPER_PARTIAL_F32) {
        *err = "unknown partial_format";
        return TAPER_EINVAL;
    }
    return TAPER_OK;
}

namespace {

constexpr int64_t kPieceCostTokens = 200;   // what one more piece of a cut sequence costs, in tokens' streaming time
constexpr int64_t kOnePerUnitLossPct = 3;   // what one workgroup per compute unit instead of two costs, percent
constexpr double kTokensPerMergedRow = 5.0;      // see least_tokens
constexpr int kBriefTokens = 128;            // private segments that are priced as a single wave's work, in steps of up to
constexpr int64_t kBriefShareTokens = 700;   // so many tokens per share,
constexpr int64_t kBriefItemCost = 160;      // at so much (see Cost::brief)
constexpr double kMergeLaunchFromUs = 10.5;   // see merges_after
constexpr int64_t kSaturatingShareTokens = 350;  // shares of fewer tokens are over before the memory system is saturated
constexpr int64_t kRoomyShareTokens = 128;       // with so few there are shares to spare (one holds 256 as a rule): prefixes may be cut finer
constexpr int64_t kLongShareTokens = 2000;       // from here on private work holds back beside shared-prefix work (see private_item in the kernels)

struct Segment {
    int32_t seq0, n_branch, page0, n_tokens, kind;
    int32_t ends_seq = 0;  // private: the last tokens of its sequence in plan order (whoever streams them usually merges)
    int32_t whole_seq = 0;  // private: the sequence's whole context
    int32_t siblings = 0;   // shared: this and the next siblings - 1 segments stream the same prefix (one request, cut into sub-groups)
    int32_t pct = 100;      // cost of a token, percent of a private one's
};

// Cost model of a workgroup share, in units of one private token's streaming time: an item of
// n tokens costs fixed + n * pct / 100 (pct: its segment's), `fixed` covering what an item costs beyond
// streaming its tokens (query load, pipeline fill, partial rows, arrival, merges).
struct Cost {
    int64_t fixed;
    int64_t merge = 0;  // extra cost of the item that ends a sequence: it arrives last as a rule and merges the partials
    int64_t per_branch = 0;  // further fixed cost for each of a shared item's branches
    // Short private segments are run by single waves, four side by side (order_solo_items), and merged by whoever comes later: they cost
    // no merge, and are not worth a claim from the pool; with it an item of the whole workgroup is 320 to 384.  (Where steps have no such
    // merge cost, or short shares, `fixed` is 128: 160 is more than that, and still the better price there: with 128 35 random steps take 0.8 % more
    // on average, from 5 % less to 9 % more.)  In steps of long shares that is not
    // so: their chain of dependent loads is several times as long on a saturated machine, and whoever finishes early takes them from the
    // pool (411 sequences of 12 to 22 tokens beside 8 requests of 4 to 6 branches 65 -> 41 us per layer, 30 requests of 14 branches of 1 or 2 tokens 66 -> 43,
    // 35 requests of 32 tokens and 9 branches of 11 30 -> 21; 100 us per layer where shares have 3600 tokens and 212 short
    // branches, 110 with this price).
    int brief_tokens = 0;
    bool brief(const Segment& s) const { return s.n_tokens <= brief_tokens; }
    int64_t item(const Segment& s) const { return fixed + per_branch * s.n_branch; }
    int64_t piece(const Segment& s) const { return brief(s) ? kBriefItemCost : fixed; }  // of a private segment
    // of the item that ends a sequence: nothing where that is its only one, as a rule when it is much shorter than a share
    int64_t end(const Segment& s, int64_t share) const { return s.ends_seq && !brief(s) && !(brief_tokens && s.whole_seq && s.n_tokens * 4 <= share) ? merge : 0; }
};

// Cuts `segs` into workgroup shares of about `quota` cost units, at multiples of `blk` tokens
// from each segment's start: shares are filled one after the other, a segment going on into the
// next share where one is full.  Appends items (tagged with part ids starting at part_id0) and
// returns the number of shares used.
int partition_fill(const std::vector<Segment>& segs, int64_t quota, int blk, const Cost cost, int part_id0,
                   std::vector<taper_work_item>* items) {
    int64_t total_tokens = 0;
    for (const Segment& s : segs) total_tokens += s.n_tokens;
    if (total_tokens == 0) return 0;
    quota = std::max<int64_t>(1, quota);
    const int64_t blk_cost = blk;
    int part = 0;
    int64_t fill = 0;
    for (const Segment& s : segs) {
        const int64_t fixed = cost.piece(s);
        // a piece is only worth an item of its own if its streaming outweighs the item's fixed cost
        const int64_t min_blocks = std::max<int64_t>(1, (fixed + blk_cost - 1) / blk_cost);
        const int64_t cap = std::max<int64_t>(1, (quota - fixed) / blk_cost);  // blocks of an item with a share to itself
        int64_t remaining = (s.n_tokens + blk - 1) / blk, off = 0;  // blocks
        while (remaining > 0) {
            const int64_t room = (quota - fill - fixed) / blk_cost;  // blocks that still fit this share
            if (fill > 0 && room < remaining && room < min_blocks) {        // start the next share instead
                ++part;
                fill = 0;
                continue;
            }
            int64_t take = std::min(remaining, std::max<int64_t>(room, 1));
            // A sequence much shorter than a share is not cut: cutting would turn one item that needs no
            // partial rows at all into two with a merge.  It goes whole into this share if at least half of
            // it fits, else into the next.
            if (s.whole_seq && off == 0 && take < remaining && remaining * 4 <= cap) {
                if (fill > 0 && room * 2 < remaining) {
                    ++part;
                    fill = 0;
                    continue;
                }
                take = remaining;
            }
            if (remaining - take > 0 && remaining - take < min_blocks) take = remaining;  // no sliver left behind
            taper_work_item it;
            std::memset(&it, 0, sizeof it);
            it.seq0 = s.seq0;
            it.n_branch = s.n_branch;
            it.page0 = s.page0 + (int32_t)(off * blk / 16);
            it.n_tokens = (int32_t)std::min<int64_t>(take * blk, s.n_tokens - off * blk);
            it.kind = s.kind;
            it.part = part_id0 + part;
            items->push_back(it);
            fill += fixed + take * blk_cost;
            off += take;
            remaining -= take;
            if (remaining == 0) fill += cost.end(s, quota);
            if (fill >= quota) {
                ++part;
                fill = 0;
            }
        }
    }
    return fill > 0 ? part + 1 : part;
}

// A prefix of n tokens cut into k items takes n / k tokens' time to stream and k times its R query rows to merge.  The sum is least at
// some k * k = kTokensPerMergedRow * n / R.  Where one workgroup makes the merges (the last to arrive, for every branch of the
// request), a token costs a shared workgroup alone 20 ns, a row and item 7 ns (5 branches x 16 heads: 109 us for 195 items), and 4
// was the best constant (24000 tokens of 2 / 5 / 12 branches on one kv head of 16 query heads 33 / 46.5 / 81 us; 2.9: 32 / 49 / 85; 8: 38 /
// 48 / 83).  A step of so many items that this decides its cut has its merges in a launch of their own (all of 76 among 1250 random steps),
// where a row is cheaper: with 5 instead of 4 the mixed batch on one kv head takes 20.3 instead of 21.0, 13 branches x 8 heads of 25000 tokens 29.6 / 31.4, 13 x 16 of 4900 25.2 / 27.6; 8 would
// give another 2 to 12 % to requests of ten branches and take 4 % from narrow ones.
int64_t least_tokens(const Segment& s, int gqa) {
    return (int64_t)std::sqrt((double)s.n_tokens * s.n_branch * gqa / kTokensPerMergedRow);
}

// The same for items with a large fixed cost (shared-prefix items).  A segment that does not
// fit what is left of the current share tops it up (if that is worth an item); what then
// remains, if it is more than one share, is cut into equal items with a share each rather than
// into full shares and a remainder (which would either be a short item paying the full fixed
// cost or make the last item much longer than the others).  The last of those items is
// `tail_discount` blocks shorter: the workgroup that finishes a shared prefix usually finds the
// request's branches complete and has to merge them all.
int partition_even(const std::vector<Segment>& segs, int gqa, int64_t quota, int blk, const Cost cost, int64_t tail_discount,
                   bool crowded, bool apart, int part_id0, std::vector<taper_work_item>* items) {
    quota = std::max<int64_t>(1, quota);
    int part = 0;
    int64_t fill = 0, blk_cost = 1;
    auto emit = [&](const Segment& s, int64_t off, int64_t take) {
        taper_work_item it;
        std::memset(&it, 0, sizeof it);
        it.seq0 = s.seq0;
        it.n_branch = s.n_branch;
        it.page0 = s.page0 + (int32_t)(off * blk / 16);
        it.n_tokens = (int32_t)std::min<int64_t>(take * blk, s.n_tokens - off * blk);
        it.kind = s.kind;
        it.part = part_id0 + part;
        items->push_back(it);
        fill += cost.item(s) + take * blk_cost;
    };
    auto close = [&]() {
        if (fill > 0) ++part;
        fill = 0;
    };
    for (size_t si = 0; si < segs.size(); ++si) {
        const Segment& s = segs[si];
        if (apart) close();
        blk_cost = std::max<int64_t>(1, (int64_t)blk * s.pct / 100);
        const int64_t min_blocks = std::max<int64_t>(1, (cost.item(s) + blk_cost - 1) / blk_cost);
        // blocks of an item with a share to itself
        const int64_t cap = std::max({min_blocks, (quota - cost.item(s)) / blk_cost, least_tokens(s, gqa) / blk});
        if (s.siblings >= 2 && (!crowded || (cost.item(s) + (int64_t)s.n_tokens * s.pct / 100) * 2 >= quota)) {
            // Sub-groups of one request read the same pages.  They get the same cuts, every item a share of its
            // own and therefore the launch's start as its start, in workgroups next to each other: the sub-groups
            // then stream the prefix in step, and what the first one fetched is still in the L2 of the XCD (one
            // per kv head) when the others ask for it.  Shares that come out short take from the pool; where the sub-groups
            // alone would have most of the grid's shares (`crowded`), only items that fill half of one are placed so (26
            // requests of 33 branches and prefixes of 106 to 421 tokens: 52 shares of one such item each left 12 for 220000 private
            // tokens, 297 us; 238 this way.  12 requests of 33 branches and 36 to 64 tokens, 36 of 128 shares: 194 with a share each, 204
            // without; 64 branches 277, and 290 if a whole share were asked for).
            close();
            const int64_t blocks = (s.n_tokens + blk - 1) / blk;
            const int64_t spread = blocks + tail_discount;
            const int64_t k = blocks <= cap + min_blocks / 2 ? 1 : std::min(blocks, std::max<int64_t>(1, (spread + cap - 1) / cap));
            int64_t remaining = blocks, off = 0;
            for (int64_t i = 0; i < k; ++i) {
                int64_t take = spread / k + (i < spread % k ? 1 : 0);
                take = i + 1 < k ? std::max<int64_t>(1, std::min(take, remaining - (k - 1 - i))) : remaining;
                for (int j = 0; j < s.siblings; ++j) {
                    emit(segs[si + j], off, take);
                    close();
                }
                off += take;
                remaining -= take;
            }
            si += s.siblings - 1;
            continue;
        }
        int64_t remaining = (s.n_tokens + blk - 1) / blk, off = 0;  // blocks
        int64_t room = (quota - fill - cost.item(s)) / blk_cost;    // blocks that still fit the current share
        if (fill > 0 && room < remaining && room < min_blocks) {    // not worth an item: start the next share
            close();
            room = cap;
        }
        if (remaining > room && fill > 0) {  // top the current share up
            emit(s, 0, room);
            close();
            off = room;
            remaining -= room;
        }
        if (remaining <= cap + min_blocks / 2) {  // one item; the next segment may top its share up
            emit(s, off, remaining);
            if (fill >= quota) close();
            continue;
        }
        const int64_t spread = remaining + tail_discount;
        const int64_t k = std::min(remaining, std::max<int64_t>(1, (spread + cap - 1) / cap));  // (the discount is no block to cut)
        for (int64_t i = 0; i < k; ++i) {
            int64_t take = spread / k + (i < spread % k ? 1 : 0);
            take = i + 1 < k ? std::max<int64_t>(1, std::min(take, remaining - (k - 1 - i))) : remaining;
            emit(s, off, take);
            close();
            off += take;
            remaining -= take;
        }
    }
    close();
    return part;
}

// Shares are filled in order, and one whose last sequence is not cut comes out shorter or longer than the quota.  Dealt out again,
// the longest item to the emptiest share, they differ by less than an item.  Taken where the fullest share shrinks by 2 %, in steps
// without shared-prefix work (512 sequences of 32 to 512 tokens 101.2 -> 99.0 us, 13 short
// sequences and two of 14000 tokens in six pieces each 37.5 -> 35.6; beside shared work as often 4 % slower as faster).
void level_shares(int n_parts, const Cost& cost, std::vector<taper_work_item>* items) {
    if (n_parts < 2) return;
    const auto price = [&](const taper_work_item& it) { return (it.n_tokens <= cost.brief_tokens ? kBriefItemCost : cost.fixed) + it.n_tokens; };
    std::vector<int64_t> load(n_parts, 0);
    for (const taper_work_item& it : *items) load[it.part] += price(it);
    const int64_t most = *std::max_element(load.begin(), load.end());
    std::vector<taper_work_item> dealt(*items);
    std::stable_sort(dealt.begin(), dealt.end(), [](const taper_work_item& x, const taper_work_item& y) { return x.n_tokens > y.n_tokens; });
    std::vector<std::pair<int64_t, int>> heap(n_parts);  // (load, share), the emptiest first
    for (int q = 0; q < n_parts; ++q) heap[q] = {0, q};
    const auto later = std::greater<std::pair<int64_t, int>>();
    for (taper_work_item& it : dealt) {
        std::pop_heap(heap.begin(), heap.end(), later);
        heap.back().first += price(it);
        it.part = heap.back().second;
        std::push_heap(heap.begin(), heap.end(), later);
    }
    const int64_t least_most = std::max_element(heap.begin(), heap.end())->first;
    if (least_most * 100 > most * 98) return;
    std::stable_sort(dealt.begin(), dealt.end(), [](const taper_work_item& x, const taper_work_item& y) { return x.part < y.part; });
    *items = std::move(dealt);
}

// What a step that ends all at once takes, in us, if its merges are made in the attention launch: 4 to the first block, the longest
// share's chain of blocks (a shared one's by the row tiles of its waves) and query rows, and `rounds` of its longest merge.  Least squares over
// 318 random steps of 3 rounds and more below 350 tokens per share: within 11 % of the measured time for half of them, 18 % rms (15 below 25 us; those
// below 13 us read 10 % long).  With 1.4 us for every shared block, as before its scores were made a block ahead, half were within 13 %, 23 % rms.
double expected_us(const taper_attn_config& cfg, const HostPlan& p, int64_t rounds) {
    const int g = cfg.n_q_heads / cfg.n_kv_heads, shared_block = cfg.head_dim == 128 ? 32 : 64;
    const auto blocks = [](int n, int per) { return (double)((n + per - 1) / per); };
    const double block_us = cfg.head_dim == 128 ? 1 : 0.8;
    double longest = 0;
    for (int q = 0; q < p.n_parts_shared + p.n_parts_private; ++q) {
        double us = 0, wave[4] = {0, 0, 0, 0};
        const int solo_end = p.part_start[q] + (p.part_turn[q] >> kPartSoloShift);
        for (int i = p.part_start[q]; i < p.part_start[q + 1]; ++i) {
            const taper_work_item& it = p.items[i];
            const int k = i - p.part_start[q];
            if (it.kind == 0) us += (it.n_branch * g <= 4 * 16 ? 0.85 : it.n_branch * g <= 8 * 16 ? 1.3 : 1.55) * block_us * blocks(it.n_tokens, shared_block) + 0.04 * it.n_branch * g;
            else if (i < solo_end) wave[k / 4 % 2 ? 3 - k % 4 : k % 4] += 1.2 * blocks(it.n_tokens, kPrivateBlockTokens);
            else us += 0.6 * blocks(it.n_tokens, 4 * kPrivateBlockTokens);
        }
        longest = std::max(longest, us + *std::max_element(wave, wave + 4));
    }
    return 4 + longest + (cfg.head_dim == 128 ? 1.25 : 1.05) * rounds;
}

// Whether the step's merges are a launch of their own (merge_kernel) instead of being made by whoever delivers a sequence's last
// partial.  What counts is the longest merge that one workgroup would make alone at the end: a shared item's branches side by
// side, eight at a time, 8 rows each, in rounds of 8 entries (4 of fp32 rows); such a round is 1 to 1.7 us.  The launch costs 2 to 3 us, its
// boundary and three trips to memory, and the merged rows' way through the caches, about 3 MB per us.  Attention calls on the same cuts,
// merged behind / inside, us.  Steps that end all at once (below 350 tokens per share): 5 rounds and more 0.60 of the time on average over 169 random
// ones (11.5 / 39.5 at best, 12.2 / 11.7 the only one slower); 3 and 4 rounds 0.85 over 149, 26 of them slower (12.0 / 19.4 at best, 46.6 / 35.8 at worst).
// Longer ones, where most merges are hidden behind other workgroups' streaming: 18 of 37 of 3 and 4 rounds slower (119.5 / 105.1 at worst) and 19 faster
// (46.4 / 51.4 at best).
// A launch is also 3 us of the host's time (a call 8.5 instead of 5.9), which a step of several layers with a small launch between them waits for where the
// layers are short.  With merges inside, the same 318 steps by what a call takes: below 10, 10 to 12, 12 to 15, 15 to 18 and 18 to 22 us a call alone gains 0.9,
// 1.4, 2.6, 3.5 and 5.2 us by the launch; a loop of four layers loses 3.9, 3.1 and 0.9 us per layer, then gains 1.1 and 3.7.  kMergeLaunchFromUs lies
// where the one side's gain grows past the other's loss: of the 8 steps expected to take less, calls would gain 0 to 3.5 us and loops lose
// 3.2 to 4.7; of the 5 from there to 12, calls gain 0.7 to 4.8 and loops lose 0 to 3.6.
bool merges_after(const taper_attn_config& cfg, const HostPlan& p, bool ends_at_once) {
    const int g = cfg.n_q_heads / cfg.n_kv_heads, per_round = cfg.partial_format == TAPER_PARTIAL_F32 ? 4 : 8;
    int64_t rounds = 0, rows = 0;
    for (int s = 0; s < p.n_seqs; ++s) rows += (int64_t)(p.merge_start[s + 1] - p.merge_start[s]) * cfg.n_q_heads;
    for (const taper_work_item& it : p.items) {
        int most = 0;
        for (int s = it.seq0; s < it.seq0 + it.n_branch; ++s) most = std::max(most, p.merge_start[s + 1] - p.merge_start[s]);
        const int turns = it.kind != 0 ? 1 : (it.n_branch <= 4 ? 1 : (it.n_branch + 7) / 8) * ((g + 7) / 8);
        rounds = std::max<int64_t>(rounds, (int64_t)turns * ((most + per_round - 1) / per_round));
    }
    const int64_t bytes = rows * cfg.head_dim * (cfg.partial_format == TAPER_PARTIAL_F32 ? 4 : 2);
    if (rounds < (ends_at_once ? 3 : 5) || rounds * 3 <= 6 + bytes / 2500000) return false;  // (in units of half a us)
    return !ends_at_once || expected_us(cfg, p, rounds) >= kMergeLaunchFromUs;
}

// Workgroup w of share q works on kv head (w + turn[q]) mod n_kv_heads.  Workgroups are dealt to the XCDs in turn, and the
// XCDs do not read equally fast (the odd ones were 12 to 15 % behind in launches of shared work alone), so the
// shares take turns: every XCD then has workgroups of every head, and each head's pool evens the XCDs out.  The
// sub-groups of one request keep the turn of the first: the same head of the same chunk stays on one XCD, whose
// L2 they share it in.
void plan_part_turns(const taper_attn_config& cfg, const int32_t* branch_group, HostPlan* p) {
    const int n_parts = p->n_parts_shared + p->n_parts_private;
    p->part_turn.resize(n_parts);
    for (int q = 0; q < n_parts; ++q) {
        p->part_turn[q] = q % std::min(cfg.n_kv_heads, kPartTurnMask + 1);
        if (q == 0 || q >= p->n_parts_shared || p->part_start[q - 1] == p->part_start[q] || p->part_start[q] == p->part_start[q + 1]) continue;
        const taper_work_item &a = p->items[p->part_start[q - 1]], &b = p->items[p->part_start[q]];
        if (a.seq0 != b.seq0 && branch_group[a.seq0] == branch_group[b.seq0] && a.page0 == b.page0 && a.n_tokens == b.n_tokens)
            p->part_turn[q] = p->part_turn[q - 1];
    }
}

// Short private items of a share are run by single waves, four side by side, without barriers: a workgroup's four waves get one block
// each of a 128-token item and nothing of a shorter one, all latency and no streaming, and a share of many of them was a chain of
// item ends (30 requests of 8 to 11 branches of up to 11 tokens each, 8 items of 3 us one after the other: 30.5 us, 22.6; 9 requests of 34
// branches of up to 32 tokens 48.6, 27.5; 289 sequences of 2 to 8 tokens 6.9 either way).  They come before the
// share's other items, longest first, and are dealt to the waves.  An item of one block is a single wave's work in any case; fewer
// than four longer ones leave waves idle, which costs more than the barriers from 256 tokens on.
// Partials only in steps of short shares (`partials`): on a saturated machine an item's chain of dependent loads takes several times as long,
// and a wave has one item at a time (57 shared shares of 3200 tokens beside 69 short branches in 7 private ones: 80 us per layer, 84 to 86).
void order_solo_items(int n_seqs, int most_tokens, bool partials, HostPlan* p) {
    if (most_tokens <= 0) return;
    std::vector<int32_t> pieces;
    if (!partials) {
        pieces.assign(n_seqs, 0);
        for (const taper_work_item& it : p->items)
            for (int b = 0; b < it.n_branch; ++b) pieces[it.seq0 + b]++;
    }
    std::vector<taper_work_item> rest;
    for (int q = p->n_parts_shared; q < p->n_parts_shared + p->n_parts_private; ++q) {
        const auto first = p->items.begin() + p->part_start[q], end = p->items.begin() + p->part_start[q + 1];
        const auto solo = [&](const taper_work_item& it, int limit) { return it.n_tokens <= limit && (partials || pieces[it.seq0] == 1); };
        int upto[3] = {0, 0, 0};
        const int limits[3] = {most_tokens, std::min(most_tokens, 256), std::min(most_tokens, kPrivateBlockTokens)};
        for (auto it = first; it != end; ++it)
            for (int k = 0; k < 3; ++k) upto[k] += solo(*it, limits[k]);
        const int k = upto[0] >= 4 ? 0 : upto[1] >= 2 ? 1 : 2;
        if (upto[k] == 0) continue;
        if (end - first > 1) {
            rest.clear();
            auto to = first;
            for (auto it = first; it != end; ++it) {
                if (!solo(*it, limits[k])) rest.push_back(*it);
                else *to++ = *it;
            }
            std::sort(first, to, [](const taper_work_item& x, const taper_work_item& y) {
                return x.n_tokens != y.n_tokens ? x.n_tokens > y.n_tokens : x.seq0 != y.seq0 ? x.seq0 < y.seq0 : x.page0 < y.page0;
            });
            std::copy(rest.begin(), rest.end(), to);
        }
        p->part_turn[q] |= (int)std::min<int64_t>(upto[k], (1 << (31 - kPartSoloShift)) - 1) << kPartSoloShift;
    }
}

// The start records: the first item of a share and the pages its waves ask for first (past the item's last page: that one).  A private
// item's block is two pages, and wave w takes blocks w and w + 4; of a solo item it takes blocks 0 and 1.  Of a shared item every wave
// stages its part of pages 0 to 7 at head_dim 128, and pages w, w + 4, ... at 64.
// A step on one kv head has some 490 shares, so every word is written once and an item not once for each wave unless some share needs it.
// (From the call to the image on the device such a plan takes 56.7 us; 62.5 with a record of 80 bytes for each wave, 157 KB, and 47 without records.)
void make_starts(const taper_attn_config& cfg, HostPlan* p) {
    const int n_parts = p->n_parts_shared + p->n_parts_private;
    bool four = false;
    for (int q = 0; q < n_parts; ++q) four |= p->part_turn[q] >> kPartSoloShift > 1;
    p->start_bytes = four ? kStartBytesFour : kStartBytesOne;
    p->starts.resize((size_t)n_parts * p->start_bytes / sizeof(StartWords));
    for (int q = 0; q < n_parts; ++q) {
        char* to = (char*)p->starts.data() + (size_t)q * p->start_bytes;
        ShareStart s;
        s.first = p->part_start[q];
        s.end = p->part_start[q + 1];
        s.turn = p->part_turn[q] & ((1 << kPartSoloShift) - 1);
        s.n_solo = p->part_turn[q] >> kPartSoloShift;
        std::memset(s.more, 0, sizeof s.more);
        std::memset(s.page, 0, sizeof s.page);
        if (s.first == s.end) {
            std::memset(s.item, 0, sizeof s.item);
            std::memcpy(to, &s, p->start_bytes);
            continue;
        }
        const auto row_of = [&](const taper_work_item& it) { return p->block_table.data() + (size_t)it.seq0 * p->bt_stride + it.page0; };
        const auto last_of = [](const taper_work_item& it) { return (it.n_tokens + 15) / 16 - 1; };
        const taper_work_item& it = p->items[s.first];
        const int32_t* row = row_of(it);
        const int last = last_of(it);
        for (int w = 0; w < (four ? 4 : 1); ++w) s.item[w] = p->items[s.first + (w < s.n_solo ? w : 0)];
        if (it.kind == 0) {
            for (int w = 0; w < 4; ++w)
                for (int i = 0; i < 4; ++i) s.page[w][i] = row[std::min(cfg.head_dim == 128 ? i : 4 * i + w, last)];
            for (int i = 0; i < 4; ++i) s.more[i] = row[std::min(4 + i, last)];
        } else if (s.n_solo == 0) {
            for (int w = 0; w < 4; ++w)
                for (int i = 0; i < 4; ++i) s.page[w][i] = row[std::min(2 * (w + 4 * (i / 2)) + i % 2, last)];
        } else {
            for (int w = 0; w < 4; ++w)
                for (int i = 0; i < 4; ++i) {
                    const bool solo = w < s.n_solo;
                    const taper_work_item& own = p->items[s.first + (solo ? w : 0)];
                    s.page[w][i] = row_of(own)[std::min(solo ? i : 2 * (w + 4 * (i / 2)) + i % 2, last_of(own))];
                }
        }
        std::memcpy(to, &s, p->start_bytes);
    }
}

}  // namespace

int build_host_plan(const taper_attn_config& cfg, int n_seqs, const int32_t* block_table, int bt_row_stride,
                    const int32_t* branch_group, const int32_t* prefix_len, const int32_t* suffix_len,
                    int64_t n_pool_pages, const taper_plan_options* opts, HostPlan* out, std::string* err) {
    if (!suffix_len || n_seqs < 1) {
        *err = "null argument";
        return TAPER_EINVAL;
    }
    std::vector<int32_t> seg_start(n_seqs + 1);
    for (int s = 0; s <= n_seqs; ++s) seg_start[s] = s;  // one private segment per sequence
    return build_host_plan_segments(cfg, n_seqs, block_table, bt_row_stride, branch_group, prefix_len, seg_start.data(),
                                    suffix_len, n_pool_pages, opts, out, err);
}

static int build_for_grid(const taper_attn_config& cfg, int n_seqs, const int32_t* block_table, int bt_row_stride,
                          const int32_t* branch_group, const int32_t* prefix_len, const int32_t* seg_start,
                          const int32_t* seg_len, int64_t n_pool_pages, const taper_plan_options* opts,
                          HostPlan* out, std::string* err) {
    int st = validate_config(cfg, err);
    if (st != TAPER_OK) return st;
    if (!block_table || !branch_group || !prefix_len || !seg_start || !out) {
        *err = "null argument";
        return TAPER_EINVAL;
    }
    if (n_seqs < 1 || bt_row_stride < 1 || n_pool_pages < 1) {
        *err = "n_seqs, bt_row_stride and n_pool_pages must be positive";
        return TAPER_EINVAL;
    }
    if (n_pool_pages > (int64_t)1 << 31) {
        *err = "n_pool_pages exceeds the int32 page id range";
        return TAPER_EINVAL;
    }
    const int P = cfg.page_size;
    const int g = cfg.n_q_heads / cfg.n_kv_heads;
    int target_wgs = opts && opts->target_workgroups > 0 ? opts->target_workgroups : 512;
    const bool share_prefix = opts ? opts->share_prefix != 0 : true;
    // A shared item holds up to 12 row tiles.  At head_dim 64 requests are cut at 8 unless asked otherwise: a line from a kernel
    // that ran only one workgroup of more per compute unit, which no longer holds (146 to 149 VGPRs, two workgroups).  One
    // item of up to 12 tiles instead measures 79.6 us against 94.6 at 33 branches of 4 query heads, 93 against 99 at 40, 104 against
    // 111 at 48; with 8 query heads 75 against 84 at 17 branches, but 80.8 against 78.4 at 20 and 83 against 81 at 24.
    // 64: per-branch flags of the shared kernel.
    const int hard_cap = std::min(64, std::max(2, kMaxRowTilesPerItem * 16 / g));
    int cap_branches = std::min(hard_cap, std::max(2, (cfg.head_dim == 128 ? kMaxRowTilesPerItem : 8) * 16 / g));
    if (opts && opts->max_branches_per_item > 0) cap_branches = std::max(1, std::min(hard_cap, opts->max_branches_per_item));

    HostPlan& p = *out;
    p = HostPlan();
    p.n_seqs = n_seqs;
    p.bt_stride = bt_row_stride;
    p.n_pool_pages = n_pool_pages;
    p.prefix_len.assign(prefix_len, prefix_len + n_seqs);
    // private segments: CSR per sequence, lengths, and the block-table entry each one starts at
    if (seg_start[0] != 0) {
        *err = "seg_start[0] must be 0";
        return TAPER_EINVAL;
    }
    for (int s = 0; s < n_seqs; ++s)
        if (seg_start[s + 1] < seg_start[s]) {
            *err = fmt("sequence %lld: seg_start must not decrease", s);
            return TAPER_EINVAL;
        }
    if (seg_start[n_seqs] > 0 && !seg_len) {
        *err = "null argument";
        return TAPER_EINVAL;
    }
    p.seg_start.assign(seg_start, seg_start + n_seqs + 1);
    p.seg_len.assign(seg_len, seg_len + seg_start[n_seqs]);
    p.seg_page0.assign(seg_start[n_seqs], 0);
    p.suffix_len.assign(n_seqs, 0);
    p.ctx_len.resize(n_seqs);
    p.n_prefix_pages.resize(n_seqs);
    p.n_suffix_pages.resize(n_seqs);
    p.block_table.assign((size_t)n_seqs * bt_row_stride, -1);

    // ---- validation + per-sequence integers
    for (int s = 0; s < n_seqs; ++s) {
        const int64_t pl = prefix_len[s];
        int64_t sl = 0, nsp = 0;
        if (pl < 0) {
            *err = fmt("sequence %lld: negative length", s);
            return TAPER_ELEN;
        }
        const int64_t npp = (pl + P - 1) / P;
        for (int k = seg_start[s]; k < seg_start[s + 1]; ++k) {
            if (seg_len[k] < 0) {
                *err = fmt("sequence %lld: negative length", s);
                return TAPER_ELEN;
            }
            p.seg_page0[k] = (int32_t)std::min<int64_t>(npp + nsp, INT32_MAX);
            sl += seg_len[k];
            nsp += (seg_len[k] + P - 1) / P;
        }
        if (pl + sl < 1) {
            *err = fmt("sequence %lld: empty context", s);
            return TAPER_ELEN;
        }
        if (pl + sl > (1 << 30)) {
            *err = fmt("sequence %lld: context too long", s);
            return TAPER_ELEN;
        }
        p.suffix_len[s] = (int32_t)sl;
        if (npp + nsp > bt_row_stride) {
            *err = fmt("sequence %lld: needs %lld block-table entries, row has %lld", s, npp + nsp, bt_row_stride);
            return TAPER_ELEN;
        }
        p.ctx_len[s] = (int32_t)(pl + sl);
        p.n_prefix_pages[s] = (int32_t)npp;
        p.n_suffix_pages[s] = (int32_t)nsp;
        const int32_t* row = block_table + (size_t)s * bt_row_stride;
        for (int j = 0; j < npp + nsp; ++j) {
            if (row[j] < 0 || row[j] >= n_pool_pages) {
                *err = fmt("sequence %lld entry %lld: page %lld outside the pool", s, j, row[j]);
                return TAPER_EBLOCK;
            }
            p.block_table[(size_t)s * bt_row_stride + j] = row[j];
        }
        p.tokens_logical += pl + sl;
    }
    // ---- request CSR
    for (int s = 0; s < n_seqs; ++s) {
        if (s == 0) {
            if (branch_group[0] != 0) {
                *err = "branch_group must start at 0";
                return TAPER_EGROUP;
            }
            p.group_start.push_back(0);
        } else if (branch_group[s] == branch_group[s - 1] + 1) {
            p.group_start.push_back(s);
        } else if (branch_group[s] != branch_group[s - 1]) {
            *err = fmt("sequence %lld: branch_group must be non-decreasing in steps of 1", s);
            return TAPER_EGROUP;
        }
    }
    p.n_groups = (int)p.group_start.size();
    p.group_start.push_back(n_seqs);
    for (int gi = 0; gi < p.n_groups; ++gi) {
        const int a = p.group_start[gi], b = p.group_start[gi + 1];
        for (int s = a + 1; s < b; ++s) {
            if (prefix_len[s] != prefix_len[a]) {
                *err = fmt("sequence %lld: prefix_len differs from its request's first member", s);
                return TAPER_EGROUP;
            }
            if (std::memcmp(block_table + (size_t)s * bt_row_stride, block_table + (size_t)a * bt_row_stride,
                            sizeof(int32_t) * p.n_prefix_pages[a]) != 0) {
                *err = fmt("sequence %lld: prefix pages differ from its request's first member", s);
                return TAPER_EGROUP;
            }
        }
    }

    // ---- segments of KV to stream
    std::vector<Segment> shared, priv;
    for (int gi = 0; gi < p.n_groups; ++gi) {
        const int a = p.group_start[gi], b = p.group_start[gi + 1], B = b - a;
        const int pl = prefix_len[a];
        p.tokens_unique += pl;
        if (pl > 0) {
            if (B >= 2 && share_prefix) {
                const int n_sub = (B + cap_branches - 1) / cap_branches;
                const size_t first = shared.size();
                for (int k = 0; k < n_sub; ++k) {  // balanced sub-groups of at most cap_branches
                    const int lo = a + (int)((int64_t)B * k / n_sub), hi = a + (int)((int64_t)B * (k + 1) / n_sub);
                    if (hi - lo >= 2)
                        shared.push_back({lo, hi - lo, 0, pl, 0});
                    else if (hi - lo == 1)
                        priv.push_back({lo, 1, 0, pl, 1});
                }
                if (shared.size() - first >= 2 && !(opts && opts->scatter_sub_groups)) shared[first].siblings = (int32_t)(shared.size() - first);
            } else {
                for (int s = a; s < b; ++s) priv.push_back({s, 1, 0, pl, 1});
            }
        }
        for (int s = a; s < b; ++s) {
            p.tokens_unique += p.suffix_len[s];
            for (int k = seg_start[s]; k < seg_start[s + 1]; ++k)
                if (seg_len[k] > 0) priv.push_back({s, 1, p.seg_page0[k], seg_len[k], 1});
            if (!priv.empty() && priv.back().seq0 == s) priv.back().ends_seq = 1;
        }
    }

    {  // private segments that are their sequence's whole context
        std::vector<int32_t> pieces(n_seqs, 0);
        for (const Segment& s : shared)
            for (int b = 0; b < s.n_branch; ++b) pieces[s.seq0 + b] += 2;
        for (const Segment& s : priv) pieces[s.seq0] += 1;
        for (Segment& s : priv) s.whole_seq = pieces[s.seq0] == 1;
    }

    // ---- workgroup shares: both kinds run in one launch and should finish together.  A share's time is, to a few
    // percent, a sum over its items of a fixed part (first loads, rows of several branches to store, arrival,
    // merges) and a part per token.  Which kind's tokens cost more depends on what bounds the launch:
    //  * shares of some hundred tokens and more keep the memory system saturated, and a workgroup gets a slice of it.  A
    //    shared workgroup then takes 0.6 to 0.65 of the time of a private one per token (20.6 against 31.8 us per 1024
    //    tokens in the mixed batch, least squares over its shares) and 13.8 us per item, a private one 6.1 us.  Measured
    //    optimum of the launch, with the pool evening out the rest: 70 to 90 % per token for items of up to 4 row tiles.
    //  * shorter ones are over before that, and what counts is a workgroup's own chain of blocks: 15, 23 and 29 us per 1024 tokens for
    //    a shared one of up to 4, 8 and 12 row tiles, 9 for a private one, whose four waves each have a block in flight.  180 % for
    //    all and 32 per branch where the grid is full (140 / 220 / 300 and 20 there: the mixed batch on one kv head, 232 tokens per share, 19.5
    //    us either way, two steps of 233 and 236 4 and 7 % slower); 140 / 220 / 300 and 20 below kRoomyShareTokens, where finer cuts cost no other
    //    work its share.  (Against 180 and 32, with the loops as they are: 2 prefixes of 500 tokens and 19 branches 28.6 -> 17.8 us, 2 of 736 and 41
    //    31.7 -> 24.5, 10 of 402 and 10 24.2 -> 18.7; 11 of 300 to 600 and 8 24.8 -> 27.5, whose rows are then too many for a merge launch of their own.)
    const int parts_total = std::max(1, target_wgs / cfg.n_kv_heads);
    int64_t tok_listed = 0, tok_priv = 0;
    for (const Segment& s : shared) tok_listed += s.n_tokens;
    for (const Segment& s : priv) tok_priv += s.n_tokens;
    tok_listed += tok_priv;
    const int64_t share_tokens = tok_listed / parts_total;
    const bool latency_bound = share_tokens < kSaturatingShareTokens;
    bool roomy = share_tokens < kRoomyShareTokens;  // (until the cut says otherwise)
    p.long_shares = share_tokens >= kLongShareTokens;
    // An item of more than 4 row tiles gives waves two or three tiles, and a block's chain 0.74 or 0.89 us instead of 0.47: it no
    // longer keeps up with its slice of a saturated memory system.  (80 / 100 / 120 / 140 %, 8 requests of 2048 to 8192 tokens
    // beside 16 serial ones, us: 4 branches, 2 tiles, 76.0 / 76.5 / 76.3 / 77.1; 10, 5 tiles, 101.7 / 95.0 / 94.0 / 94.6; 18, 9 tiles,
    // 130.5 / 116.9 / 114.9 / 114.8; 24, 12 tiles, 159 / 138 / 134 / 135.)  Sub-groups of one request find part of their tokens in the L2
    // (64 branches, 11 tiles: 270 at 80 to 110 %, 275 at 120; 48, 12 tiles: 221 / 216 / 217 / 218), but a request has all its
    // sub-groups' items end at once, which short shares do not even out (110 / 120 / 140 / 160 / 180 %, 5 such requests beside 48 serial
    // ones: 40 branches, 1269 tokens per share, 82.8 / 75.2 / 75.3 / 75.7 / 76.6; 60, 837, 72.5 / 63.9 / 63.9 / 65.2 / 66.3; 60, 1340, 89.3 /
    // 89.7 / 89.3 / 85.9 / 84.2; 60, 2011, 116 / 116 / 112 / 112 / 112; 60, 2683, 140.5 / 140.4 / 142.9 / 143.8 / 143.8).
    auto shared_pct = [&](const Segment& s, bool sub_group) -> int32_t {
        if (opts && opts->shared_cost_pct > 0) return opts->shared_cost_pct;
        if (latency_bound && !roomy) return 180;
        if (latency_bound) return s.n_branch * g <= 4 * 16 ? 140 : s.n_branch * g <= 8 * 16 ? 220 : 300;
        return s.n_branch * g <= 4 * 16 ? 80 : !sub_group ? 120 : p.long_shares ? 110 : 160;
    };
    Cost cost_shared = {};
    const auto price_shared = [&] {  // the sum of all
        cost_shared = {opts && opts->shared_item_cost > 0 ? opts->shared_item_cost : (latency_bound ? 60 : 450), 0,
                       opts && opts->shared_item_cost > 0 ? 0 : (roomy ? 20 : latency_bound ? 32 : 0)};
        int64_t sum = 0;
        for (size_t i = 0; i < shared.size(); ++i) {
            Segment& s = shared[i];  // (the sub-groups of a request follow each other: same pages, another first sequence)
            auto same_request = [&](size_t j) { return j < shared.size() && branch_group[shared[j].seq0] == branch_group[s.seq0]; };
            s.pct = shared_pct(s, same_request(i + 1) || (i > 0 && same_request(i - 1)));
            sum += cost_shared.item(s) + (int64_t)s.n_tokens * s.pct / 100;
        }
        return sum;
    };
    // (a caller's own costs are taken as they are, and what no single wave will run is priced as the workgroup's)
    const bool own_costs = opts && (opts->private_item_cost > 0 || opts->private_merge_cost != 0);
    const int solo_tokens = opts && opts->solo_item_tokens != 0 ? std::max(0, opts->solo_item_tokens) : 512;
    const int brief_tokens = share_tokens <= kBriefShareTokens && !own_costs ? std::min(kBriefTokens, solo_tokens) : 0;
    const Cost cost_priv = {opts && opts->private_item_cost > 0 ? opts->private_item_cost : (shared.empty() || latency_bound ? 128 : 192),
                            opts && opts->private_merge_cost != 0 ? std::max(0, opts->private_merge_cost)
                                                                  : (shared.empty() ? 0 : 192),
                            0, brief_tokens};
    const int64_t shared_tail_discount = 3;  // blocks: about what merging a request's branches costs
    int64_t cost_of_shared = price_shared(), cost_total = cost_of_shared;
    for (const Segment& s : priv) {
        cost_total += cost_priv.piece(s) + s.n_tokens + cost_priv.end(s, share_tokens);
    }
    // ---- the pool: private tokens no share owns.  No cost model predicts the shares' running times
    // to better than some ten percent (the XCDs are not equally fast, page placement matters, and of two workgroups
    // on a compute unit the one dispatched first is served first: with equal long shares it leaves at half the
    // launch), so the shares are cut short and every workgroup that finishes its share takes items
    // from the pool until it is empty.  The longer the shares, the larger the differences and the less a pool
    // item's fixed cost weighs: a quarter of the private tokens for shares of up to 2048 tokens, rising to 60 % at
    // 5120.  (25 / 40 / 60 %: mixed batch, 1900 tokens per share, 83.1 / 83.9 / 85.8 us; 8 requests of 64 branches, 5400 per
    // share, 335 / 330 / 267, where what changes is how often the sub-groups' prefixes are cut; 640 sequences, 19000 per share, 798 /
    // 790 / 796.)  Without shared-prefix work the shares are alike and cutting a sequence costs more than the balance gains; and
    // where latency bounds the launch a claim's round trip is as much as it evens out (26.7 us without, 26.0 with 30 %, 28.6 with 25 % and
    // the constants of longer shares, mixed batch on one kv head).
    const int pool_default = shared.empty() || latency_bound
                                 ? 0
                                 : (int)(25 + 35 * std::min<int64_t>(3072, std::max<int64_t>(0, share_tokens - 2048)) / 3072);
    const int pool_pct = opts && opts->pool_pct != 0 ? std::max(0, std::min(90, opts->pool_pct)) : pool_default;
    const int pool_item_opt = opts && opts->pool_item_tokens > 0 ? opts->pool_item_tokens : 0;
    std::vector<Segment> pool;
    {
        int64_t want = tok_priv * pool_pct / 100;
        size_t left = priv.size();
        for (size_t i = priv.size(); i-- > 0 && want >= kPrivateBlockTokens;) {
            Segment& s = priv[i];
            if (cost_priv.brief(s) && !(opts && opts->pool_pct > 0)) continue;  // (a claim would cost more than the item)
            const bool last = shared.empty() && left == 1;  // (a launch has a workgroup per share: one stays)
            if (s.n_tokens <= want + kPrivateBlockTokens && !last) {  // the whole segment
                want -= s.n_tokens;
                cost_total -= cost_priv.piece(s) + s.n_tokens + cost_priv.end(s, share_tokens);
                pool.push_back(s);
                s.n_tokens = 0;
                --left;
            } else {  // its tail, from a block boundary
                const int keep = (int)((s.n_tokens - want + kPrivateBlockTokens - 1) / kPrivateBlockTokens * kPrivateBlockTokens);
                if (keep < s.n_tokens) {
                    pool.push_back({s.seq0, s.n_branch, s.page0 + keep / 16, s.n_tokens - keep, s.kind, s.ends_seq, 0});
                    cost_total -= s.n_tokens - keep + cost_priv.end(s, share_tokens);
                    s.whole_seq = 0;
                    s.n_tokens = keep;
                    s.ends_seq = 0;
                }
                want = 0;
            }
        }
        std::reverse(pool.begin(), pool.end());
        priv.erase(std::remove_if(priv.begin(), priv.end(), [](const Segment& s) { return s.n_tokens == 0; }), priv.end());
    }
    // A small step is not cut as finely as the grid allows: below a few hundred tokens per share the
    // time goes into the item ends.  Nor is a sequence cut into very many partials: up to 32 are one trip of the merge launch and 64 two; half
    // as many beside shared prefixes, whose own cuts come on top (one sequence of 15000 tokens on 2 kv heads 12.4 -> 10.2 us, 12 requests of
    // 14 branches or reduced and 27000 tokens on one 32.5 -> 23.8 against 16 partials at most; two small steps the other way, 28.6 -> 30.1 and
    // 15.6 -> 16.4).  Where the merges stay inside the launch as well: 26.4 -> 24.4, 34.0 -> 30.3, 34.4 -> 31.5; two even, and two of ten or
    // eleven sequences of some 3000 tokens on one kv head 9.4 -> 9.8 and 9.5 -> 9.9 (a third round of merges).
    int64_t longest = 0;
    for (const Segment& s : priv) longest = std::max<int64_t>(longest, s.n_tokens);
    const int64_t min_share =
        (opts && opts->min_share_tokens > 0 ? opts->min_share_tokens : std::max<int64_t>(256, longest / (shared.empty() ? 64 : 32))) + cost_priv.fixed;
    int64_t quota = 0;
    // Never more shares than asked for: an extra one would run after all the others.  The quota is raised by small steps until that is
    // so: by as many at once as the excess suggests, and halved back between the last one that was too low and the first that is not.
    int64_t sub_groups = 0;
    for (const Segment& s : shared) sub_groups += s.siblings;
    const bool crowded = sub_groups * 2 > parts_total;
    // Where shares are over early and there are enough of them a prefix gets one of its own (two of 60 tokens one after the other: 11.6 us, 8.4).
    const auto cut = [&](int64_t q) {
        const bool apart = roomy && (int64_t)shared.size() * 2 <= parts_total;
        p.items.clear();
        p.n_parts_shared = partition_even(shared, g, q, kSharedBlockTokens, cost_shared, shared_tail_discount, crowded, apart, 0, &p.items);
        p.n_parts_private = partition_fill(priv, q, kPrivateBlockTokens, cost_priv, p.n_parts_shared, &p.items);
        return p.n_parts_shared + p.n_parts_private <= parts_total || q >= cost_total * 2 + 4096;
    };
    const auto search = [&] {
        quota = std::max<int64_t>(std::max<int64_t>(kSharedBlockTokens, min_share), (cost_total + parts_total - 1) / parts_total);
        std::vector<int64_t> tried = {quota};  // the steps
        auto step = [&](size_t i) {
            while (tried.size() <= i) tried.push_back(tried.back() + std::max<int64_t>(16, tried.back() / 256));
            return tried[i];
        };
        size_t below = 0, at = 0;
        while (!cut(step(at))) {
            below = at++;
            const int64_t enough = tried[below] * (p.n_parts_shared + p.n_parts_private) / parts_total;
            while (step(at) < enough) ++at;
        }
        bool current = true;
        while (at - below > 1) {
            const size_t mid = (below + at) / 2;
            current = cut(step(mid));
            (current ? at : below) = mid;
        }
        quota = step(at);
        if (!current) cut(quota);
    };
    search();
    // Finer cuts pay while shared workgroups have a compute unit each.  Two side by side share its matrix cores and issue slots, and at head_dim 128
    // their chains of blocks become longer than the coarser ones: beyond half of the shares the prices are those of fuller grids.  us, with
    // the one and the other: 8 requests of 33 branches 32.2 / 26.7 (51 % of the shares), 7 of 49 33.8 / 29.0 (52 %), 10 of 40 36.2 / 29.3 (54 %), 8 of 17 36.8 / 30.8 (59 %), 10
    // of 20 39.9 / 30.2 (69 %), 12 of 49 47.1 / 47.2 (80 %); below it 8 of 33 22.8 / 24.3 (38 %), 11 of 49 24.2 / 29.1 (41 %), 3 of 17 17.3 / 20.4 (48 %), 7 of 49 25.8 / 28.9
    // (50 %), one the other way (7 of 40, 49 %, 25.9 / 24.0).  At head_dim 64 a block is half the work: 9 of 17 15.0 / 19.6 (52 %).
    if (roomy && cfg.head_dim == 128 && p.n_parts_shared * 2 > parts_total) {
        roomy = false;
        cost_total -= cost_of_shared;
        cost_total += price_shared();
        search();
    }
    if (shared.empty()) level_shares(p.n_parts_private, cost_priv, &p.items);
    const int n_parts = p.n_parts_shared + p.n_parts_private;
    p.part_start.assign(n_parts + 1, 0);
    for (const taper_work_item& it : p.items) p.part_start[it.part + 1]++;
    for (int i = 0; i < n_parts; ++i) p.part_start[i + 1] += p.part_start[i];
    plan_part_turns(cfg, branch_group, &p);
    // size of the pool's items: a quarter of a share, between 512 and 1536 tokens, unless the caller says otherwise
    const int pool_item_tokens = std::max<int>(
        kPrivateBlockTokens,
        (pool_item_opt ? pool_item_opt : (int)std::min<int64_t>(1536, std::max<int64_t>(512, quota / 4))) / kPrivateBlockTokens * kPrivateBlockTokens);
    for (const Segment& s : pool) {  // pool items follow the shares' items; their `part` is n_parts
        const int k = (s.n_tokens + pool_item_tokens - 1) / pool_item_tokens;
        const int piece = ((s.n_tokens + k - 1) / k + kPrivateBlockTokens - 1) / kPrivateBlockTokens * kPrivateBlockTokens;
        for (int off = 0; off < s.n_tokens; off += piece) {
            taper_work_item it;
            std::memset(&it, 0, sizeof it);
            it.seq0 = s.seq0;
            it.n_branch = 1;
            it.page0 = s.page0 + off / 16;
            it.n_tokens = std::min(piece, s.n_tokens - off);
            it.kind = 1;
            it.part = n_parts;
            p.items.push_back(it);
        }
    }
    p.n_pool_items = (int)p.items.size() - p.part_start[n_parts];
    // longest first: the launch's last claims are then the shortest items
    std::stable_sort(p.items.begin() + p.part_start[n_parts], p.items.end(),
                     [](const taper_work_item& x, const taper_work_item& y) { return x.n_tokens > y.n_tokens; });

    order_solo_items(n_seqs, solo_tokens, share_tokens <= kBriefShareTokens, &p);

    // ---- partial rows and merge map
    int64_t rows = 0;
    p.merge_start.assign(n_seqs + 1, 0);
    for (taper_work_item& it : p.items) {
        if (it.n_tokens < 1) {  // the kernels index pages by an item's last token: never launched
            *err = "internal error: a work item without tokens";
            return TAPER_EINVAL;
        }
        // (the merge addresses partial rows by 32-bit byte offsets: fp32 rows of a step stay below 2^31 bytes)
        if ((rows + (int64_t)it.n_branch * cfg.n_q_heads) * cfg.head_dim * 4 > INT32_MAX) {
            *err = "too many partial rows";
            return TAPER_EINVAL;
        }
        it.part_base = (int32_t)rows;
        const int rph = it.n_branch * g;
        if (it.kind == 0) p.max_row_tiles_shared = std::max(p.max_row_tiles_shared, (rph + 15) / 16);
        for (int b = 0; b < it.n_branch; ++b) p.merge_start[it.seq0 + b + 1]++;
        rows += (int64_t)rph * cfg.n_kv_heads;
    }
    p.n_partial_rows = rows;
    for (int s = 0; s < n_seqs; ++s) p.merge_start[s + 1] += p.merge_start[s];
    p.merge.resize(p.merge_start[n_seqs]);
    std::vector<int32_t> filled(p.merge_start.begin(), p.merge_start.end() - 1);
    for (const taper_work_item& it : p.items)
        for (int b = 0; b < it.n_branch; ++b) p.merge[filled[it.seq0 + b]++] = {it.part_base + b * g, it.n_branch * g};
    p.merge_after = merges_after(cfg, p, latency_bound);
    for (taper_work_item& it : p.items) {
        it.merge0 = p.merge_start[it.seq0];
        // a private item that is its sequence's whole context needs no partial rows: the kernel writes the result
        if (it.kind == 1 && p.merge_start[it.seq0 + 1] - p.merge_start[it.seq0] == 1) it.kind = 2;
    }
    for (int q = p.n_parts_shared; q < n_parts; ++q)
        for (int i = p.part_start[q]; i < p.part_start[q] + (p.part_turn[q] >> kPartSoloShift); ++i) {
            if (p.items[i].kind == 2) p.items[i].kind = 3;
            else p.part_turn[q] |= kPartSoloPartials;
        }
    return TAPER_OK;
}

// Cutting a sequence costs: every piece writes partial rows, announces them, and one workgroup reads them all back
// (three dependent trips through a loaded memory system, some 200 tokens' streaming time per piece).  A step
// without shared-prefix work whose shares are short is therefore also cut for half the grid -- one workgroup per
// compute unit instead of two, which alone reads 1 to 4 % slower -- and that plan is taken when it saves enough
// pieces to pay for it.  (32 requests of 1024-4096 tokens: 86 pieces become 54 and the launch 2.5 % faster;
// 32 equal requests: no piece at all, 5-10 % faster; a large step has few pieces per share either way.)
static void take_fewer_pieces(const taper_attn_config& cfg, int n_seqs, const int32_t* block_table, int bt_row_stride,
                              const int32_t* branch_group, const int32_t* prefix_len, const int32_t* seg_start,
                              const int32_t* seg_len, int64_t n_pool_pages, const taper_plan_options* opts, HostPlan* out) {
    if (!opts || opts->small_step_grid <= 0) return;
    const int grid = opts->target_workgroups > 0 ? opts->target_workgroups : 512;
    const int parts_full = std::max(1, grid / cfg.n_kv_heads);
    if (out->n_parts_shared != 0 || out->n_pool_items != 0 || out->n_parts_private < parts_full || parts_full < 2) return;
    auto pieces = [](const HostPlan& h) {
        int64_t n = 0;
        for (const taper_work_item& it : h.items) n += it.kind == 1;
        return n;
    };
    const int64_t pieces_full = pieces(*out);
    if (pieces_full * kPieceCostTokens * 100 <= out->tokens_unique * kOnePerUnitLossPct) return;  // cannot pay even if all went
    taper_plan_options half = *opts;
    half.target_workgroups = grid / 2;
    HostPlan alt;
    std::string err2;
    if (build_for_grid(cfg, n_seqs, block_table, bt_row_stride, branch_group, prefix_len, seg_start, seg_len, n_pool_pages,
                       &half, &alt, &err2) != TAPER_OK)
        return;
    if ((pieces_full - pieces(alt)) * kPieceCostTokens * 100 > out->tokens_unique * kOnePerUnitLossPct) *out = std::move(alt);
}

int build_host_plan_segments(const taper_attn_config& cfg, int n_seqs, const int32_t* block_table, int bt_row_stride,
                             const int32_t* branch_group, const int32_t* prefix_len, const int32_t* seg_start,
                             const int32_t* seg_len, int64_t n_pool_pages, const taper_plan_options* opts,
                             HostPlan* out, std::string* err) {
    int st = build_for_grid(cfg, n_seqs, block_table, bt_row_stride, branch_group, prefix_len, seg_start, seg_len,
                            n_pool_pages, opts, out, err);
    if (st != TAPER_OK) return st;
    take_fewer_pieces(cfg, n_seqs, block_table, bt_row_stride, branch_group, prefix_len, seg_start, seg_len, n_pool_pages, opts, out);
    make_starts(cfg, out);
    return TAPER_OK;
}

void resolve_slots_host(const HostPlan& p, int P, int64_t* slots, int64_t stride) {
    for (int s = 0; s < p.n_seqs; ++s) {
        const int32_t* row = p.block_table.data() + (size_t)s * p.bt_stride;
        for (int64_t t = 0; t < stride; ++t) {
            int64_t v = -1;
            if (t < p.ctx_len[s]) {
                if (t < p.prefix_len[s]) {
                    v = (int64_t)row[t / P] * P + t % P;
                } else {
                    int64_t j = t - p.prefix_len[s];
                    int k = p.seg_start[s];
                    while (j >= p.seg_len[k]) j -= p.seg_len[k++];
                    v = (int64_t)row[p.seg_page0[k] + j / P] * P + j % P;
                }
            }
            slots[(size_t)s * stride + t] = v;
        }
    }
}

}  // namespace taper
