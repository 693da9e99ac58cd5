// Host side of the attention launch: which work items a call's queries and caches become, in which order.  No device code
// (a test compiles this file on its own).
#pragma once
#include <algorithm>
#include <utility>
#include <vector>

// Wavefronts per workgroup, 32 stacked query rows each.  Eight (two per SIMD) share each K / V tile, which halves the DMA into
// LDS; four leave twice the blocks (see plan_attention for when).
constexpr int ATT_WAVES = 8, ATT_WAVES_SMALL = 4;
constexpr int ATT_KEYS = 64;   // keys per tile
constexpr int ATT_MAX_PARTS = 16;
constexpr int ATT_SPLIT_SLOTS = 384;       // slots of the split buffer (a block that finds no free slots stays whole)
constexpr int ATT_MIN_PART_TILES = 6;      // a part is worth a workgroup and its share of the merge from about 400 keys; every row of a
                                           // block must see keys of each part: its rows span at most 256 positions, 5 tiles
constexpr int ATT_MIN_SPLIT_TILES = 16;    // no block of the call is split unless the longest walks at least 1024 keys

struct AttnItem {
    int req;
    int kvh;
    int qblock;  // block of 32 WAVES stacked query rows
    int nkb;     // number of 64-key tiles this block must visit (tiles [0, nkb), or [kb0, nkb) for a part of a split block)
    int kb0;     // first tile of this part (0 unless the block's key range is split)
    int slot;    // -1: the workgroup finishes the block and writes the output; >= 0: it leaves an unnormalised partial
                 // result in this slot of the split buffer (see AttnPartial) for attn_merge_kernel
    int pad0_, pad1_;
};
struct AttnMergeItem {
    int req;
    int kvh;
    int qblock;
    int n_parts;
    int slot0;  // the parts' slots are slot0 .. slot0 + n_parts - 1
    int pad0_, pad1_, pad2_;
};

struct AttnRequest {
    int T, P;   // rows of the call, tokens cached before it
    bool operator==(const AttnRequest& o) const { return T == o.T && P == o.P; }
};
struct AttnPlanSettings {
    int n_cu;           // compute units
    int split;          // RS_ATTN_SPLIT: 0 decided here, 1 nothing is cut, n > 1 parts of every block
    bool plain_order;   // RS_ATTN_ORDER=plain: blocks that share a compute unit stay in heaviest-first order
};
struct AttnPlan {
    int waves = ATT_WAVES;
    int cost = 0;   // estimated duration, in tiles (0: nothing was weighed)
    std::vector<AttnItem> items;
    std::vector<AttnMergeItem> merges;
};

// The plan of the layer before, in a call of several layers: good for the next one if its caches have the same lengths.
struct AttnPlanCache {
    std::vector<AttnRequest> reqs;   // empty: no plan yet
    AttnPlan plan;
};

// Where a block of n tiles is cut: in equal parts of at most `cap` tiles, in parts of exactly `cap` and a rest (!even), or (cap 0)
// not at all.
struct AttnCut {
    int cap = 0;
    bool even = true;
    int parts = 0;   // > 0: this many parts (RS_ATTN_SPLIT)
    // number of parts (1: whole) and the tiles of every part but the last (0: equal parts)
    std::pair<int, int> of(int n) const {
        int p = 1, step = 0;
        if (parts > 0) {
            p = std::min(parts, n / ATT_MIN_PART_TILES);
        } else if (cap > 0 && even) {
            p = std::min(std::min((n + cap - 1) / cap, n / ATT_MIN_PART_TILES), ATT_MAX_PARTS);
        } else if (cap > 0) {
            const int full = n / cap, rest = n - full * cap;
            p = rest < ATT_MIN_PART_TILES ? full : full + 1;
            step = rest < ATT_MIN_PART_TILES ? 0 : cap;
        }
        return p < 2 || p > ATT_MAX_PARTS ? std::make_pair(1, 0) : std::make_pair(p, step);
    }
};

// How many of `count` such blocks of n tiles are cut when `slots` of the split buffer are taken: a block that finds no free slots
// stays whole.
inline int attn_blocks_cut(const AttnCut& cut, int n, int count, int slots) {
    const int p = cut.of(n).first;
    return p < 2 ? 0 : std::min(count, (ATT_SPLIT_SLOTS - slots) / p);
}
// End of part i of p of a block of n tiles (`step`: see AttnCut::of).
inline int attn_part_end(int n, int p, int step, int i) { return step ? std::min((i + 1) * step, n) : (int)((long)(i + 1) * n / p); }

// Heaviest first, equals in their order.
inline void attn_sort_items(std::vector<AttnItem>& items) {
    int longest = 0;
    for (const AttnItem& it : items) longest = std::max(longest, it.nkb - it.kb0);
    std::vector<int> at(longest + 2, 0);
    for (const AttnItem& it : items) ++at[it.nkb - it.kb0];
    for (int n = longest, first = 0; n >= 0; --n) {
        const int count = at[n];
        at[n] = first;
        first += count;
    }
    std::vector<AttnItem> sorted(items.size());
    for (const AttnItem& it : items) sorted[at[it.nkb - it.kb0]++] = it;
    items.swap(sorted);
}

// The estimates are in units of one key tile's time on a full chip (1.6 to 1.8 us at d = 128); the constants are fitted to kernel
// traces (the merge 6 us, and 14 us for 392 parts; a part's partial result 133 KB at d = 128).
constexpr int ATT_COST_ITEM = 2, ATT_COST_PART = 4, ATT_COST_MERGE = 4, ATT_COST_MERGE_PARTS = 36;   // per whole item, part, merge; parts per further one

// Equally long blocks (KV heads and requests repeat lengths: a few dozen groups stand for hundreds of blocks).
struct AttnGroup {
    int n, count;   // tiles of a block, blocks
};
inline std::vector<AttnGroup> attn_groups(const std::vector<AttnItem>& blocks) {   // (heaviest first)
    std::vector<AttnGroup> groups;
    for (const AttnItem& b : blocks) {
        if (groups.empty() || groups.back().n != b.nkb) groups.push_back(AttnGroup{b.nkb, 0});
        ++groups.back().count;
    }
    return groups;
}

// Estimated duration of a launch of these blocks under a cut, the items handed out longest first, one to a compute unit at a time
// and to the next as units fall free.
inline int attn_cost(const std::vector<AttnGroup>& groups, const AttnCut& cut, int n_cu) {
    if (groups.empty()) return 0;
    std::vector<int> items((size_t)groups[0].n + ATT_COST_PART + 1, 0);   // items by cost
    int slots = 0;
    long sum = 0;
    const auto add = [&](int cost, int count) {
        items[cost] += count;
        sum += (long)cost * count;
    };
    for (const AttnGroup& g : groups) {
        const auto [p, step] = cut.of(g.n);
        const int k = attn_blocks_cut(cut, g.n, g.count, slots);
        if (k < g.count) add(g.n + ATT_COST_ITEM, g.count - k);
        if (k == 0) continue;
        for (int i = 0, first = 0; i < p; ++i) {
            const int end = attn_part_end(g.n, p, step, i);
            add(end - first + ATT_COST_PART, k);
            first = end;
        }
        slots += k * p;
    }
    std::vector<int> units((size_t)(sum / n_cu) + items.size() + 1, 0);   // compute units by load; the least load only grows
    units[0] = n_cu;
    int least = 0, end = 0;
    for (int cost = (int)items.size() - 1; cost > 0; --cost)
        for (int left = items[cost]; left > 0;) {
            while (units[least] == 0) ++least;
            const int k = std::min(left, units[least]);
            units[least] -= k;
            units[least + cost] += k;
            end = std::max(end, least + cost);
            left -= k;
        }
    return end + (slots ? ATT_COST_MERGE + slots / ATT_COST_MERGE_PARTS : 0);
}

// A call's blocks of 32 `waves` stacked rows, heaviest first, whole key ranges.
inline std::vector<AttnItem> attn_blocks(const std::vector<AttnRequest>& reqs, int group, int kv_heads, int waves) {
    std::vector<AttnItem> blocks;
    const int rows = 32 * waves;
    for (int r = 0; r < (int)reqs.size(); ++r) {
        const int n = (int)(((long)reqs[r].T * group + rows - 1) / rows);
        for (int qb = 0; qb < n; ++qb) {
            const int t_max = std::min(reqs[r].T - 1, (qb * rows + rows - 1) / group);   // the block's last token
            const int nkb = (reqs[r].P + t_max + 1 + ATT_KEYS - 1) / ATT_KEYS;
            for (int c = 0; c < kv_heads; ++c) blocks.push_back(AttnItem{r, c, qb, nkb, 0, -1, 0, 0});
        }
    }
    attn_sort_items(blocks);
    return blocks;
}

// Equal parts as long as every part has a compute unit of its own: the smallest cap with at most n_cu parts.
inline AttnCut attn_even_cut(const std::vector<AttnGroup>& groups, int n_cu) {
    AttnCut c;
    int lo = ATT_MIN_PART_TILES, hi = std::max(lo, groups[0].n);
    while (lo < hi) {
        c.cap = (lo + hi) / 2;
        long parts = 0;
        for (const AttnGroup& g : groups) parts += (long)g.count * c.of(g.n).first;
        if (parts <= n_cu) hi = c.cap; else lo = c.cap + 1;
    }
    c.cap = lo;
    return c;
}

// Two blocks of four wavefronts to a compute unit (between n_cu and 2 n_cu of them, heaviest first, nothing cut): the heaviest run
// alone, the others in pairs, heavy with light, and all are there from the first clock.  A pair shares the unit until the light one
// ends, at the rate of a block of eight (289.8 us against 287.1 at d = 128, 179.4 against 183.2 at d = 64, 512 blocks of 128 rows on
// 8192 tokens); a block alone takes 0.65 (d = 128) to 0.70 (d = 64) of that per tile: ATT_COST_ALONE / 16.
constexpr int ATT_COST_ALONE = 11;
inline int attn_pairs_cost(const std::vector<AttnItem>& blocks, int n_cu) {
    const int n = (int)blocks.size(), lone = 2 * n_cu - n;
    int end = blocks[0].nkb * ATT_COST_ALONE;
    for (int k = 0; k < n - n_cu; ++k) {
        const int heavy = blocks[lone + k].nkb, light = blocks[n - 1 - k].nkb;
        end = std::max(end, 16 * light + (heavy - light) * ATT_COST_ALONE);
    }
    return (end + 15) / 16 + ATT_COST_ITEM;
}
// Their order.  On an empty chip the dispatcher hands workgroup k and workgroup k + n_cu to the same compute unit (measured: 448
// workgroups that fit two to a unit leave exactly workgroups 192 .. 255 alone on theirs).
inline void attn_place_pairs(std::vector<AttnItem>& blocks, int n_cu, int kv_heads) {
    const int n = (int)blocks.size(), paired = n - n_cu, lone = n_cu - paired;
    std::vector<AttnItem> placed(n);
    for (int k = 0; k < lone; ++k) placed[paired + k] = blocks[k];
    // (the light partners are taken from the tail in runs of one block per KV head, in the head order of the front: the blocks of a
    //  head then stay on the XCDs, workgroup index mod 8, whose L2 already holds that head's K and V)
    const bool by_head = n % kv_heads == 0 && paired % kv_heads == 0;
    for (int k = 0; k < paired; ++k) {
        placed[k] = blocks[lone + k];
        placed[n_cu + k] = by_head ? blocks[n - kv_heads * (k / kv_heads + 1) + k % kv_heads] : blocks[n - 1 - k];
    }
    blocks.swap(placed);
}

constexpr int ATT_SMALL_WALK_TILES = 64;
constexpr int ATT_SMALL_PART_TILES = 24;

// The call's work items.  One workgroup of eight wavefronts fills a compute unit, so a launch lasts as long as the fullest unit:
// key ranges are cut where that ends the launch sooner, and the parts of a cut block are combined by attn_merge_kernel.
// Measured at the 7B shape, attention step, nothing cut (RS_ATTN_SPLIT=1) -> planned: 64 rows on 2048 cached tokens 38 -> 21 us, 250
// on 8192: 162 -> 49, 1000 on 12000: 272 -> 169; 16 requests, 2048 rows, caches of 0 to 12288 tokens 206 -> 174.  4096 rows on 28672
// (1024 blocks) stay whole.
// Calls too small to fill the chip even with every key range cut as finely as it may be take blocks of four wavefronts: twice the
// workgroups, and a wavefront that has its SIMD to itself (attention step with eight and with four, 64 rows on 2048 cached tokens,
// 7B shape: 24.4 and 20.5 us; tiny shape, 128 rows on 384: 14.0 and 11.4).  So do calls whose small blocks have, in equal parts one
// to a compute unit, ATT_SMALL_PART_TILES or fewer (blocks of eight leave half the parts, of twice the bytes; with longer walks
// their one fetch per 256 rows counts for more).  Eight and four, us, with the tiles of the longest small part: 7B, 250 rows on 2000
// (9) 29.7 and 27.0, three requests of 83 to 150 rows on 500 to 3000 (12) 34.1 and 28.4, 512 on 1536 (16) 33.6 and 33.0, 700 on 700
// (22) 33.3 and 32.2, 250 on 8192 (33) 48.0 and 51.6; 12 / 2 heads, 512 on 4000 (15) 33.2 and 29.8; 72B, 250 on 2000 (18) 40.9 and
// 39.6, 128 on 8000 (32) 48.2 and 49.7; 32 / 8 heads of 64, 250 on 2000 (9) 20.2 and 18.3, on 8000 (33) 32.1 and 33.4.
// So do calls of more small blocks than compute units, but no more than two to each, where the pairs of attn_pairs_cost end sooner:
// the blocks of a prompt's first chunks differ in length, and cutting them costs more than pairing.  Attention step, us, blocks of
// eight planned as above -> pairs: 7B, 2048 rows on 0 tokens 55.0 -> 46.7 (in heaviest-first order 50.4), on 2000 101 -> 93, on 6144
// 198 -> 193; 32 / 8 heads of 64, 2048 rows on 0: 40.9 -> 34.0, on 2000: 77.6 -> 65.0.
// And calls of more small blocks than that whose walks have at most ATT_SMALL_WALK_TILES: with two blocks on a unit one's first loads
// and last stores pass behind the other's products, which counts most where walks are short and blocks many; with long walks the
// fetches count again.  Eight and four, us, with the longest walk: 72B, 16 requests of 200 rows on 200 tokens (7) 96.5 and 79.6, 32 of
// 100 on 1000 (18) 175 and 154, 1200 rows on 0 (19) 47.0 and 42.0, 3000 on 0 (47) 175 and 165, 3000 on 1000 (63) 303 and 282, 4096 on 0
// (64) 289 and 286, 2048 on 8000 (157) 526 and 539; 7B, 4096 on 0 (64) 123.5 and 123.6, on 1000 (80) 171 and 177.
inline AttnPlan plan_attention(const AttnPlanSettings& s, const std::vector<AttnRequest>& reqs, int group, int kv_heads) {
    AttnPlan plan;
    long n_small = 0, most = 0;   // small blocks, parts they could be cut into
    for (const AttnRequest& r : reqs) {
        const long blocks = ((long)r.T * group + 32 * ATT_WAVES_SMALL - 1) / (32 * ATT_WAVES_SMALL) * kv_heads;
        const long tiles = ((long)r.P + r.T + ATT_KEYS - 1) / ATT_KEYS;
        n_small += blocks;
        most += blocks * (tiles < ATT_MIN_SPLIT_TILES ? 1 : std::min<long>(tiles / ATT_MIN_PART_TILES, ATT_MAX_PARTS));
    }
    if (n_small == 0) return plan;
    std::vector<AttnItem> blocks;
    bool small = most <= s.n_cu;
    if (small || n_small <= s.n_cu) blocks = attn_blocks(reqs, group, kv_heads, ATT_WAVES_SMALL);
    if (!small && n_small <= s.n_cu) {
        const std::vector<AttnGroup> g = attn_groups(blocks);
        const AttnCut even = g[0].n >= ATT_MIN_SPLIT_TILES ? attn_even_cut(g, s.n_cu) : AttnCut{};
        small = (g[0].n + even.of(g[0].n).first - 1) / even.of(g[0].n).first <= ATT_SMALL_PART_TILES;
    }
    if (small) plan.waves = ATT_WAVES_SMALL;
    else blocks = attn_blocks(reqs, group, kv_heads, ATT_WAVES);

    if (s.split <= 1 && (s.split == 1 || blocks[0].nkb < ATT_MIN_SPLIT_TILES) && n_small <= s.n_cu) {   // (nothing to weigh)
        plan.items.swap(blocks);
        return plan;
    }
    AttnCut cut;
    const std::vector<AttnGroup> groups = attn_groups(blocks);
    const int longest = groups[0].n, n = (int)blocks.size();
    if (s.split <= 1) plan.cost = attn_cost(groups, cut, s.n_cu);
    if (s.split > 1) {
        cut.parts = s.split;
    } else if (s.split == 0 && longest >= ATT_MIN_SPLIT_TILES) {
        const auto consider = [&](AttnCut c) {
            const int cost = attn_cost(groups, c, s.n_cu);
            if (cost < plan.cost) {
                plan.cost = cost;
                cut = c;
            }
        };
        // (1) equal parts, one to a compute unit
        if (n < s.n_cu) consider(attn_even_cut(groups, s.n_cu));
        // (2) an even share for every compute unit: blocks longer than the share are cut there, the rests fill the gaps
        long work = 0;
        for (const AttnGroup& g : groups) work += (long)g.n * g.count;
        AttnCut c;
        c.even = false;
        c.cap = (int)((work + (long)n * ATT_COST_PART) * 102 / 100 / s.n_cu) + 1;
        if (c.cap >= ATT_MIN_PART_TILES && c.cap + ATT_MIN_PART_TILES <= longest) consider(c);
    }
    if (plan.waves == ATT_WAVES && s.split <= 1 && n_small > s.n_cu && (n_small <= 2 * s.n_cu || longest <= ATT_SMALL_WALK_TILES)) {
        std::vector<AttnItem> small_blocks = attn_blocks(reqs, group, kv_heads, ATT_WAVES_SMALL);
        const bool pairs = n_small <= 2 * s.n_cu;
        const int cost = pairs ? attn_pairs_cost(small_blocks, s.n_cu) : attn_cost(attn_groups(small_blocks), AttnCut{}, 2 * s.n_cu);
        if (!pairs || cost < plan.cost) {
            if (pairs && !s.plain_order) attn_place_pairs(small_blocks, s.n_cu, kv_heads);
            plan.waves = ATT_WAVES_SMALL;
            plan.cost = cost;
            plan.items.swap(small_blocks);
            return plan;
        }
    }
    if (cut.cap == 0 && cut.parts == 0) {
        plan.items.swap(blocks);
        return plan;
    }
    plan.items.reserve(blocks.size() + ATT_SPLIT_SLOTS);
    int slots = 0;
    for (const AttnItem& b : blocks) {
        if (attn_blocks_cut(cut, b.nkb, 1, slots) == 0) {
            plan.items.push_back(b);
            continue;
        }
        const auto [p, step] = cut.of(b.nkb);
        plan.merges.push_back(AttnMergeItem{b.req, b.kvh, b.qblock, p, slots, 0, 0, 0});
        AttnItem part = b;
        part.nkb = 0;
        for (int i = 0; i < p; ++i) {
            part.kb0 = part.nkb;
            part.nkb = attn_part_end(b.nkb, p, step, i);
            part.slot = slots++;
            plan.items.push_back(part);
        }
    }
    if (!plan.merges.empty()) attn_sort_items(plan.items);
    return plan;
}
