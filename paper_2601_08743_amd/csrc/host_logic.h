// Host-only logic of libtablecache, free of the HIP headers so that it also builds with a plain C++
// compiler (the sanitizer build of tests/test_host_sanitized.py): the replacement rules of the
// device table cache (paper App. A), the allocator of sequence blocks, and the planner that turns a
// batch into attention work items.  tc_host.hip is the only user in the library.
#pragma once
#include "../../include/tablecache.h"
#include "tc_types.h"

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <list>
#include <unordered_map>
#include <vector>

namespace tc {

// ------------------------------------------------------------------ replacement rules (App. A)
// Each rule answers three questions about the set of cached tables: is the request cached,
// what happens on a hit, and who goes when a miss finds the cache full.  Tables a caller has
// pinned are passed over: the victim is the rule's first choice among the others (-1: none left).
using PinMap = std::unordered_map<int32_t, int32_t>;

class Replacement {
public:
    virtual ~Replacement() {}
    virtual bool cached(int32_t id) const = 0;
    virtual void on_hit(int32_t id) = 0;
    virtual int32_t pick_victim(const PinMap &pins) const = 0;
    virtual void remove(int32_t id) = 0;
    virtual void insert(int32_t id) = 0;
    virtual size_t size() const = 0;
    virtual void tick() {}                         // called once per request, before anything else
};

// LRU: recency list, most recent at the front; the end is evicted.
class LruRule : public Replacement {
    std::list<int32_t> order_;
    std::unordered_map<int32_t, std::list<int32_t>::iterator> pos_;
public:
    bool cached(int32_t id) const override { return pos_.count(id) != 0; }
    void on_hit(int32_t id) override { order_.splice(order_.begin(), order_, pos_[id]); }
    int32_t pick_victim(const PinMap &pins) const override {
        for (auto it = order_.rbegin(); it != order_.rend(); ++it) if (!pins.count(*it)) return *it;
        return -1;
    }
    void remove(int32_t id) override { order_.erase(pos_[id]); pos_.erase(id); }
    void insert(int32_t id) override { order_.push_front(id); pos_[id] = order_.begin(); }
    size_t size() const override { return pos_.size(); }
};

// FIFO: a queue; hits leave it alone; the head is evicted, arrivals join the tail.
class FifoRule : public Replacement {
    std::list<int32_t> queue_;
    std::unordered_map<int32_t, std::list<int32_t>::iterator> pos_;
public:
    bool cached(int32_t id) const override { return pos_.count(id) != 0; }
    void on_hit(int32_t) override {}
    int32_t pick_victim(const PinMap &pins) const override {
        for (int32_t id : queue_) if (!pins.count(id)) return id;
        return -1;
    }
    void remove(int32_t id) override { queue_.erase(pos_[id]); pos_.erase(id); }
    void insert(int32_t id) override { queue_.push_back(id); pos_[id] = std::prev(queue_.end()); }
    size_t size() const override { return pos_.size(); }
};

// LFU: (frequency, timestamp) per table; smallest frequency goes, ties by smallest timestamp.
class LfuRule : public Replacement {
    struct Stat { int64_t freq, stamp; };
    std::unordered_map<int32_t, Stat> stat_;
    int64_t clock_ = 0;
public:
    void tick() override { ++clock_; }
    bool cached(int32_t id) const override { return stat_.count(id) != 0; }
    void on_hit(int32_t id) override { Stat &s = stat_[id]; s.freq += 1; s.stamp = clock_; }
    int32_t pick_victim(const PinMap &pins) const override {
        int32_t best = -1; Stat bs{0, 0};
        for (const auto &kv : stat_)
            if (pins.count(kv.first)) continue;
            else if (best < 0 || kv.second.freq < bs.freq ||
                (kv.second.freq == bs.freq && kv.second.stamp < bs.stamp)) { best = kv.first; bs = kv.second; }
        return best;
    }
    void remove(int32_t id) override { stat_.erase(id); }
    void insert(int32_t id) override { stat_[id] = Stat{1, clock_}; }
    size_t size() const override { return stat_.size(); }
};

// One request against the cache (App. A's Update(request), with pinned tables passed over): a hit
// updates the rule's bookkeeping; a miss on a full cache removes the rule's first unpinned choice
// and inserts the request.  `refused`: a miss found every cached table pinned - nothing changed
// beyond the rule's clock.
struct CacheStep { bool hit; int32_t evicted; bool refused; };
inline CacheStep cache_request(Replacement &rule, const PinMap &pins, int64_t capacity, int32_t id)
{
    rule.tick();
    if (rule.cached(id)) { rule.on_hit(id); return CacheStep{true, -1, false}; }
    int32_t evicted = -1;
    if ((int64_t)rule.size() >= capacity) {
        evicted = rule.pick_victim(pins);
        if (evicted < 0) return CacheStep{false, -1, true};
        rule.remove(evicted);
    }
    rule.insert(id);
    return CacheStep{false, evicted, false};
}

inline Replacement *make_rule(int32_t policy)
{
    if (policy == TC_POLICY_LRU) return new LruRule;
    if (policy == TC_POLICY_FIFO) return new FifoRule;
    return new LfuRule;
}

// ------------------------------------------------------------------ sequence blocks
// Blocks [first, end) of the pool belong to sequences.  Allocation always takes the lowest-numbered
// free block (the paper has no allocator; this rule makes block tables reproducible).
// One bit per block: a batch takes and gives back tens of thousands of blocks (an ordered set of ids
// cost ~100 ns for each; 25 k blocks: 0.8 ms in the stitch and 1.9 ms in the release).
class SeqBlocks {
    int64_t first_ = 0, end_ = 0;
    size_t n_free_ = 0, hint_ = 0;         // no free block below word hint_
    std::vector<uint64_t> free_;           // bit b - first: 1 = free
    uint64_t &word(int64_t b) { return free_[(size_t)(b - first_) >> 6]; }
    static uint64_t bit(int64_t k) { return uint64_t(1) << (k & 63); }
public:
    void reset(int64_t first, int64_t end)
    {
        first_ = first; end_ = end;
        n_free_ = (size_t)(end - first);
        hint_ = 0;
        free_.assign((n_free_ + 63) / 64, ~uint64_t(0));
        if (n_free_ % 64) free_.back() = bit((int64_t)n_free_) - 1;
    }
    size_t n_free() const { return n_free_; }
    bool in_range(int64_t b) const { return b >= first_ && b < end_; }
    bool allocated(int64_t b) const { return in_range(b) && !(free_[(size_t)(b - first_) >> 6] & bit(b - first_)); }
    // the n lowest free blocks in ascending order, not taken yet (n <= n_free())
    std::vector<int32_t> lowest(size_t n) const
    {
        std::vector<int32_t> out;
        out.reserve(n);
        for (size_t w = hint_; w < free_.size() && out.size() < n; ++w)
            for (uint64_t m = free_[w]; m && out.size() < n; m &= m - 1)
                out.push_back((int32_t)(first_ + (int64_t)(w * 64) + __builtin_ctzll(m)));
        return out;
    }
    void take(int32_t b)
    {
        uint64_t &w = word(b);
        const uint64_t m = bit(b - first_);
        n_free_ -= (w & m) != 0;
        w &= ~m;
        while (hint_ < free_.size() && !free_[hint_]) ++hint_;
    }
    int32_t take_lowest() { const int32_t b = lowest(1)[0]; take(b); return b; }
    void release(int32_t b)
    {
        uint64_t &w = word(b);
        const uint64_t m = bit(b - first_);
        n_free_ += (w & m) == 0;
        w |= m;
        hint_ = std::min(hint_, (size_t)(b - first_) >> 6);
    }
};

// ------------------------------------------------------------------ plan staging
// Where the next plan goes in a staging buffer of `cap` integers that uploads read asynchronously: plans
// that fit a half take the halves in turn, so that the host waits for the upload before last and not
// for the last one; a longer plan takes the whole buffer.  `parts`: the halves it covers (bit k), all of
// whose uploads must have ended before it is written, and whose event its own upload must record.
struct StageHalves {
    int next = 0;
    struct Spot { size_t at; unsigned parts; };
    static size_t half_of(size_t cap) { return (cap / 2) & ~size_t(63); }     // (uploads move whole 16-byte chunks)
    Spot place(size_t ints, size_t cap)
    {
        if (ints > half_of(cap)) return Spot{0, 3u};
        const int k = next;
        next = 1 - k;
        return Spot{(size_t)k * half_of(cap), 1u << k};
    }
};

// ------------------------------------------------------------------ the plan of one batch
// The integer plan of one batch, host copy and layout of the device copy.
struct Plan {
    bool valid = false;
    int32_t B = 0, max_blocks = 0, total_S = 0, n_stitch_blk = 0, n_items = 0, max_splits = 1, n_groups = 0, row_blocks = 1;
    int32_t longest_range = 0;  // key tiles of the longest work item (prefill)
    int64_t n_part_slots = 0;   // partial slots of the batch: by (token, partition) in kernels that keep them by row, else by (row tile, partition)
    bool pipelined = false;     // bf16, one row block per wave: the pipelined attention kernel
    bool decode = false;        // bf16, at most one new token per query: the decode kernels
    bool pingpong = false;      // bf16, 256 rows per work-group in two alternating wave groups
    int32_t part_stride = 0;    // kernels that keep partials by row: slots from token to token, 0: packed
    int32_t n_arrivals = 0;     // row tiles that may need an arrival counter (fold)
    bool fold = false;          // partials by row are combined inside the launch that makes them (else by one of its own)
    bool part_f32 = false;      // partials in fragment order are fp32 (the long-launch kernel's, by a rule of the planner), else fp16
    bool compact = false;       // planned for the least space (a batch that did not fit the static workspace otherwise)
    bool brief = false;         // bf16, 32 rows per work-group, its waves split the keys: the short-launch kernel
    bool rope = false;          // the stitch re-encodes keys by position (Sec. 4.1.1)
    std::vector<int32_t> rope_pos0;      // [B]
    std::vector<double> rope_rev_freq;   // [D/2]
    std::vector<int32_t> block_table, cu_seqlens, prefix_len, suffix_len;
    std::vector<uint8_t> block_pad;      // aliasing sequences: unused token positions per block-table entry, else empty
    std::vector<int32_t> alias_slots;    // table slots whose blocks the batch's sequences alias
    bool fixed = false;         // plan and partials live in the static workspace (tc_prefill_attn_noalloc)
    float *part = nullptr;      // split-KV partials of this plan (null: none needed)
    BatchDev dev{};
    const AttnItem *items_dev = nullptr;
    const MergeGroup *groups_dev = nullptr;
    int32_t *arrivals_dev = nullptr;
};

// What a caller may force about the attention launch (tc_set_kv_splits and friends); 0 = automatic.
struct PlanKnobs {
    int32_t forced_splits = 0;
    int32_t forced_row_blocks = 0;
    int32_t forced_attn_kernel = 0;   // 1 general, 2 pipelined, 3 decode (where it applies), 4 long launches, 5 short launches
    int32_t short_rows = kShortRows;  // rows per work item of the short-launch kernel, 0: do without that kernel
    // For callers whose workspace is fixed: floats there are for partials (0: as many as it takes), and whether to
    // plan for the least space - one partition where a kernel can, no kernel that needs more than the general one
    // unless its launch is long.
    size_t part_cap = 0;
    bool compact = false;
};

// fp32 batches: the key range of a work item, in key tiles.  A wave works through a quarter of its
// item's 32-key units one after the other at 1.9 us each for D = 64 (4096 cycles of matrix
// instructions), about one more for start and end; a CU does that for one item at 0.8 of the full rate
// or for two at half the rate each.  Items are nearly equal, so they run in rounds of 512, and what
// a launch takes is its full rounds plus the last one, however few items that holds: ranges are cut
// so that the rounds come out full.  The merge costs a launch of ~2.5 us and its traffic (up to eight ranges of heads of 64, which
// have none, 0.3 .. 1.5 us less, which the choice does not turn on).
// Measured (8 queries, 23 k keys, 8 / 2 heads of 64): 102 us against 118..127 us for one or two ranges a query.
inline int plan_f32_range(const tc_config &c, const Plan &p, int row_tile, int key_tile, size_t part_cap)
{
    const int G = c.n_q_heads / c.n_kv_heads;
    const double unit_us = 1.9 * c.head_dim / 64.0;
    int longest = 0;
    for (int i = 0; i < p.B; ++i)
        if (p.suffix_len[i] > 0) longest = std::max(longest, (p.prefix_len[i] + p.suffix_len[i] + key_tile - 1) / key_tile);
    int best_range = 0;
    double best = 1e30;
    for (int cuts = 1; cuts <= 32; ++cuts) {
        const int range = std::max(1, (longest + cuts - 1) / cuts);
        double units = 0, partial_rows = 0, item = 0;
        int64_t n = 0;
        for (int i = 0; i < p.B; ++i) {
            const int S = p.suffix_len[i];
            if (S <= 0) continue;
            const int tiles = (p.prefix_len[i] + S + key_tile - 1) / key_tile, ns = (tiles + range - 1) / range;
            const double per_wave = std::ceil(2.0 * ((tiles + ns - 1) / ns) / 4.0) + 1.0;
            const int64_t k = (int64_t)c.n_kv_heads * ((S * G + row_tile - 1) / row_tile) * ns;
            n += k;
            units += (double)k * per_wave;
            item = std::max(item, per_wave);
            if (ns > 1) partial_rows += (double)S * c.n_q_heads * ns;
        }
        if (part_cap > 0 && partial_rows * (c.head_dim + 2) > (double)part_cap) continue;
        const int64_t rest = n % 512;
        const double us = unit_us * ((double)(n / 512) * 2.0 * (units / (double)n) + (rest == 0 ? 0.0 : rest <= 256 ? 1.25 * item : 2.0 * item)) +
                          (partial_rows > 0 ? 2.5 + 2e-6 * partial_rows * c.head_dim : 0.0);
        if (us < best - 1e-9) { best = us; best_range = range; }
        if (range == 1) break;
    }
    return best_range;
}

// The short-launch kernel (32 rows per work-group, one work-group per CU, its eight waves split the
// range's 32-key units): the key range of a work item in key tiles, and what the launch takes, in us.  A
// round of work-groups costs 4.4 us and 1.6 for each unit of a wave (a round trip to memory and its
// arithmetic: the wave has one unit in flight), the merge 3.5 us and its fp32 partials, each MB of keys and
// values 0.1 us.  Ranges are only cut where the chip has CUs to spare and a KV head has at most 512 rows (16 row
// tiles that each fetch the keys; one query of 2.1 k + 140 tokens, 28 / 4 heads: 19.1 us in two ranges, 19.5 in
// the pipelined kernel), so partials stay small, and more than two rounds of work-groups are left to the
// other kernels (three: 1.04 times as fast as those, two: 1.3, one: 1.4).  Fitted to
// 740 batches (1 .. 16 queries of 350 .. 10500 prefix and 2 .. 330 new tokens, 28 / 4, 32 / 8 and 40 / 8
// heads) in 1 .. 9 ranges, all merged by a launch of its own: 8 % rms.  Up to eight ranges are combined without one, which
// saves 0.2 .. 1 us; charged 0.4 us less for it, queries of three units a wave (450 .. 700 keys) would be cut in three ranges: of 17
// such batches 15 lose 0.1 .. 0.9 us by that (one of 538 + 22 tokens, 28 / 4 heads, 9.7 us, in one range 9.0).
inline double batch_mb(const tc_config &c, const Plan &p)
{
    double tokens = 0;
    for (int i = 0; i < p.B; ++i)
        if (p.suffix_len[i] > 0) tokens += (double)p.prefix_len[i] + p.suffix_len[i];
    return tokens * c.n_kv_heads * c.head_dim * 4e-6;
}
struct BriefPlan { int range = 0; double us = 1e30; };
inline BriefPlan plan_brief(const tc_config &c, const Plan &p, int row_tile, int key_tile, int max_tiles)
{
    const int G = c.n_q_heads / c.n_kv_heads;
    auto tiles_of = [&](int i) { return (p.prefix_len[i] + key_tile - 1) / key_tile + (p.suffix_len[i] + key_tile - 1) / key_tile; };
    int longest = 0;
    for (int i = 0; i < p.B; ++i)
        if (p.suffix_len[i] > 0) longest = std::max(longest, tiles_of(i));
    BriefPlan best;
    const double mb = batch_mb(c, p);
    for (int cuts = 1; cuts <= 32; ++cuts) {
        const int range = std::max(1, (longest + cuts - 1) / cuts);
        if (range > max_tiles) continue;
        int64_t n = 0;
        double units = 0, rows_cut = 0;
        int most = 0;
        bool split = false, wide = false;
        for (int i = 0; i < p.B; ++i) {
            const int S = p.suffix_len[i];
            if (S <= 0) continue;
            const int tiles = tiles_of(i), ns = std::min((tiles + range - 1) / range, std::max(1, tiles / 2));
            const int per_wave = (2 * ((tiles + ns - 1) / ns) + 7) / 8;
            const int64_t k = (int64_t)c.n_kv_heads * ((S * G + row_tile - 1) / row_tile) * ns;
            n += k;
            units += (double)k * per_wave;
            most = std::max(most, per_wave);
            if (ns > 1) { split = true; wide = wide || S * G > 512; rows_cut += (double)S * c.n_q_heads * ns; }
        }
        if (n == 0 || n > 512 || (split && (n > 256 || wide))) break;          // (n grows with the cuts)
        const double rounds = (double)((n + 255) / 256);
        const double us = std::max(4.4 + 1.6 * most, rounds * (4.4 + 1.6 * units / (double)n)) + (split ? 3.5 + 3e-5 * rows_cut : 0.0) + 0.1 * mb;
        if (us < best.us - 1e-9) best = BriefPlan{range, us};
        if (range == 1) break;
    }
    return best;
}

// The general and the pipelined kernel (128 rows per work-group; `row_tile` 256 with two row blocks per wave): the number of
// key partitions, by a small cost model in units of one key tile of one work-group
// (~1.4 us).  The work items of one (query, KV head, partition) - a bucket - go to one XCD (they
// share its L2), so what counts is the most loaded XCD: buckets per XCD x items per bucket over
// its 32 CUs gives the work-groups per CU (a whole number while the chip is not full: 35 items
// on an XCD mean 3 CUs run two and the launch takes as long as with 64); times the key tiles per
// work-group (co-resident work-groups overlap each other's stalls: x0.7); plus a fixed start-up
// and epilogue cost; plus the merge: a launch and the partials written and read back at about
// 4 TB/s.  Fitted to split-count sweeps and per-work-group traces on c2, c3 and c5-sized batches.
// `long_launch`: the same question for the long-launch kernel (one work-group per CU; uncut items differ in length, start
// longest first and end together rather than in rounds), which goes by plan_long but by this for the type of its partials.
struct GeneralPlan { int splits = 1; double us = 1e30; };
inline GeneralPlan plan_general(const tc_config &c, const Plan &p, int row_tile, int key_tile, size_t part_cap, bool long_launch = false)
{
    const int G = c.n_q_heads / c.n_kv_heads;
    int64_t base = 0, tiles_sum = 0, n_q = 0;
    for (int i = 0; i < p.B; ++i)
        if (p.suffix_len[i] > 0) {
            base += (int64_t)c.n_kv_heads * ((p.suffix_len[i] * G + row_tile - 1) / row_tile);
            tiles_sum += long_launch ? ((int64_t)p.prefix_len[i] + p.suffix_len[i] + key_tile - 1) / key_tile
                                     : (p.prefix_len[i] + key_tile - 1) / key_tile + (p.suffix_len[i] + key_tile - 1) / key_tile;
            ++n_q;
        }
    GeneralPlan out;
    if (base == 0) return out;
    const double tiles = (double)tiles_sum / (double)n_q;
    const double items_per_bucket = (double)base / (double)(n_q * c.n_kv_heads);
    const double rows = (double)p.total_S * c.n_q_heads;
    double best = 1e30;
    for (int ns = 1; ns <= 32; ++ns) {
        if (ns > 1 && tiles / ns < 2.0) break;
        if (ns > 1 && part_cap > 0 && (double)ns * base * row_tile * (64 + 2) > (double)part_cap) break;
        const double load = std::ceil((double)n_q * c.n_kv_heads * ns / 8.0) * items_per_bucket / 32.0;
        const double per_cu = load <= 1.0 ? 1.0 : load <= 2.0 && !(long_launch && ns == 1) ? 2.0 : load;
        const double merge = ns > 1 ? 1.0 + 0.93e-4 * ns * rows : 0.0;   // fp16 partials: 264 B per row and partition
        const double cost = per_cu * (tiles / ns) * (per_cu >= 2.0 && !long_launch ? 0.7 : 1.0) + 3.0 + merge;
        if (cost < best - 1e-9) {
            best = cost;
            out.splits = ns;
            // What such a launch takes, in us, for the comparisons with the other kernels only: fitted to 710 of the batches
            // that plan_brief was fitted to (9 % rms), with the append work-groups and the traffic, which the
            // choice between partition counts does not turn on.
            out.us = 0.8 + 7.1 * per_cu + 1.44 * per_cu * (tiles / ns) * (per_cu >= 2.0 ? 0.7 : 1.0) +
                     (ns > 1 ? 1.9 + 1e-4 * ns * rows : 0.0) + 2.2 * p.total_S / 256.0 + 0.087 * batch_mb(c, p);
        }
    }
    return out;
}

// The long-launch kernel (one work-group of 256 rows per CU): the key range of a work item in key tiles, and what the launch
// takes, in us.  The row tiles of one (query, KV head, range) - a bucket - go to one XCD, the longest first to whichever has the
// least work, and there to whichever CU is free, so the launch lasts as long as that placement of them on 8 x 32 CUs: each item
// 7.8 us and 1.32 a key tile, where some query is cut 1.8 us and its partials for the merge, and 3.0 for the launch.  One range length
// for the batch: a long query is cut into more than a short one.  Tried are lengths from the longest query's down to a
// twenty-eighth of it.
// Fitted to 90 batches, and held against 150 others (1 .. 32 queries of 0.1 .. 18 k prefix and 2 .. 512 new tokens, 28 / 4, 32 / 8 and
// 40 / 8 heads) at up to 16 lengths each, with fp16 and with fp32 partials: 7.7 % rms, and of the lengths tried the choice is
// within 0.6 % of the fastest on average, 12 % at worst.  (Placed on 256 CUs alike: 1.3 %, and 40 % at worst - one query of 4.4 k
// + 400 tokens, 28 / 4 heads, in five ranges: 20 buckets of 11 items put 33 on some XCD, 59.8 us against 42.0 in four; with one
// partition count for all, taken from a batch's mean length: 11 % behind it.)
struct LongPlan { int range = 0; double us = 1e30; bool cut = false; };
inline LongPlan plan_long(const tc_config &c, const Plan &p, int row_tile, int key_tile, size_t part_cap, bool part_f32)
{
    constexpr int kCus = 256, kXcds = 8;
    constexpr int64_t kItem = 780, kTile = 132;          // 1/100 us
    const int G = c.n_q_heads / c.n_kv_heads;
    struct Query { int tiles; int64_t row_tiles, rows; };
    std::vector<Query> queries;
    int longest = 0;
    for (int i = 0; i < p.B; ++i) {
        const int64_t S = p.suffix_len[i];
        if (S <= 0) continue;
        queries.push_back(Query{(int)(((int64_t)p.prefix_len[i] + S + key_tile - 1) / key_tile), (S * G + row_tile - 1) / row_tile, S * c.n_q_heads});
        longest = std::max(longest, queries.back().tiles);
    }
    LongPlan best;
    double uncut = 0.0;                                  // with no query cut: left for 5 % or more, which the fit resolves
    struct Part { int tiles; int64_t row_tiles, buckets; };
    std::vector<Part> parts;
    struct Xcd { int64_t load; std::vector<std::pair<int64_t, int64_t>> cus; } xcds[kXcds];      // (when free, how many), the first free last
    // (the buckets of a query's KV heads are alike: they go to as many XCDs, which then are, too, and one stands for them)
    const int alike = c.n_kv_heads % 8 == 0 ? 8 : c.n_kv_heads % 4 == 0 ? 4 : c.n_kv_heads % 2 == 0 ? 2 : 1;
    int last = 0;
    for (const int tenths : {10, 12, 14, 16, 18, 20, 25, 30, 40, 50, 60, 80, 110, 150, 200, 280}) {
        const int range = std::max(2, (longest * 10 + tenths - 1) / tenths);
        if (range == last) continue;
        last = range;
        parts.clear();
        int64_t cut_rows = 0, cut_tiles = 0, total = 0;
        for (const Query &q : queries) {
            const int ns = std::max(1, std::min((q.tiles + range - 1) / range, q.tiles / 2)), len = q.tiles / ns, more = q.tiles % ns;
            if (more) parts.push_back({len + 1, q.row_tiles, (int64_t)more * c.n_kv_heads});
            parts.push_back({len, q.row_tiles, (int64_t)(ns - more) * c.n_kv_heads});
            total += q.row_tiles * c.n_kv_heads * (ns * kItem + q.tiles * kTile);
            if (ns > 1) { cut_rows += q.rows * ns; cut_tiles += q.row_tiles * c.n_kv_heads * ns; }
        }
        if (part_cap > 0 && (double)cut_tiles * row_tile * ((part_f32 ? 128 : 64) + 2) > (double)part_cap) continue;
        const double merge = cut_rows > 0 ? 1.8 + (part_f32 ? 1.45e-4 : 0.74e-4) * (double)cut_rows : 0.0;
        std::stable_sort(parts.begin(), parts.end(), [](const Part &x, const Part &y) { return x.tiles > y.tiles; });
        if (3.0 + merge + 0.01 * (double)std::max(total / kCus, kItem + parts[0].tiles * kTile) >= (uncut > 0.0 ? std::min(best.us, 0.95 * uncut) : best.us)) continue;
        for (Xcd &x : xcds) { x.load = 0; x.cus.assign(1, {0, kCus / kXcds}); }
        for (const Part &part : parts)
            for (int64_t k = 0; k < part.buckets; k += alike) {
                Xcd *x = &xcds[0];
                for (Xcd *y = x + 1; y < xcds + kXcds / alike; ++y) if (y->load < x->load) x = y;
                x->load += (part.tiles + 3) * part.row_tiles;
                for (int64_t count = part.row_tiles; count > 0;) {
                    auto &cus = x->cus;
                    const int64_t free_at = cus.back().first, n = std::min(count, cus.back().second), end = free_at + kItem + part.tiles * kTile;
                    if ((cus.back().second -= n) == 0) cus.pop_back();
                    const auto at = std::lower_bound(cus.begin(), cus.end(), end, [](const auto &c0, int64_t t) { return c0.first > t; });
                    if (at != cus.end() && at->first == end) at->second += n;
                    else cus.insert(at, {end, n});
                    count -= n;
                }
            }
        int64_t ends = 0;
        for (Xcd *x = xcds; x < xcds + kXcds / alike; ++x) ends = std::max(ends, x->cus.front().first);
        const double us = 3.0 + merge + 0.01 * (double)ends;
        if (us < best.us - 1e-9 && (uncut == 0.0 || us < 0.95 * uncut)) best = LongPlan{range, us, cut_rows > 0};
        if (cut_rows == 0 && uncut == 0.0) uncut = us;
    }
    return best;
}

// Where the split-KV partials of the fp32, decode and short-launch kernels stand.  They are kept by row: a slot, D + 2
// floats for each query head, for every (suffix token, partition), packed: a batch pays for the partitions that its
// queries have, not for its longest query's count everywhere, and a query in one range has none.
// Where a launch of its own combines them and the queries have about as many partitions each, every token has as many slots as
// the most it could need instead, so that the merge knows them without a look into a table (0.3 us); where that would be more than
// twice the slots needed, or more than the workspace holds, they are packed there as well.
// (The other bf16 kernels keep, per (cut row tile, partition, row block), 128 rows x (128 fp16 + 2 floats)
// in fragment order, or 128 fp32.)
inline void place_partials(const tc_config &c, const PlanKnobs &knobs, Plan &p, const std::vector<int32_t> &splits_of_q,
                           std::vector<AttnItem> &items)
{
    const int64_t even = (int64_t)p.max_splits * p.total_S;       // (n_part_slots: packed, so far)
    if (!p.fold && !knobs.compact && even <= 2 * p.n_part_slots &&
        (knobs.part_cap == 0 || (size_t)even * c.n_q_heads * (c.head_dim + 2) <= knobs.part_cap)) {
        p.part_stride = p.max_splits;
        p.n_part_slots = even;
    }
    std::vector<int64_t> first(p.B);
    int64_t at = 0;
    for (int i = 0; i < p.B; ++i) {
        first[i] = p.part_stride ? (int64_t)p.cu_seqlens[i] * p.part_stride : at;
        if (splits_of_q[i] > 1) at += (int64_t)p.suffix_len[i] * splits_of_q[i];
    }
    for (AttnItem &it : items)
        if (it.q >= 0) {
            it.part0 = (int32_t)first[it.q];
            it.part_stride = p.part_stride ? p.part_stride : it.n_splits;
        }
}

// Where the workspace has no room for counters of their own (PlanLayout::counters): the counter of each row tile whose ranges' partials
// are folded inside the launch is the `arrived` of its first item.  Until here `arrival` is the tile's number, below `n_tiles`.
inline void place_arrivals(std::vector<AttnItem> &items, size_t n_tiles)
{
    std::vector<int32_t> first(n_tiles, -1);
    for (size_t k = 0; k < items.size(); ++k)
        if (items[k].q >= 0 && items[k].n_splits > 1) {
            int32_t &at = first[items[k].arrival];
            if (at < 0) at = (int32_t)k;
            items[k].arrival = at;
        }
}

// Attention work list for the batch in `p` (host arrays filled in).  Items of one
// (query, KV head, split) read the same K/V; they are given work-group ids that are congruent
// modulo 8 so that they land on the same XCD and share its L2 (work-groups go to the 8 XCDs
// round-robin by id).  Holes are padded with no-op items (q = -1).
// `pipe_cap` is the number of key tiles whose block ids one work item of the kernel in question may
// keep in LDS; returns false if an item came out longer than its kernel allows (a bug: the caller
// refuses the batch rather than launch it).
inline bool plan_attention_pass(const tc_config &c, const PlanKnobs &knobs, Plan &p, std::vector<AttnItem> &items,
                                std::vector<int32_t> &splits_of_q, std::vector<MergeGroup> &groups,
                                int general_cap, bool &cap_bound)
{
    const PlanKnobs *ctx = &knobs;
    cap_bound = false;
    items.clear();                                      // a second pass starts from nothing
    groups.clear();
    const int G = c.n_q_heads / c.n_kv_heads;
    const bool bf16 = c.dtype == TC_BF16;
    const int KT = bf16 ? kAttnKeys : kF32Keys;
    p.decode = false;
    p.pingpong = p.part_f32 = false;
    p.brief = false;
    p.n_part_slots = 0;
    p.n_groups = p.part_stride = p.n_arrivals = 0;
    p.fold = false;
    p.compact = ctx->compact;
    // Decode step: every query brings at most one new token, so a KV head has only G rows and the
    // work is reading K and V once.  The decode kernels split the keys of a (query, KV head) over
    // the four waves of a work-group and over `ns` work-groups.  A work-group holds a CU (its ring of
    // tiles fills the LDS), and what a launch of this kind costs is how its loads get going and
    // drain, once per round of work-groups: so the ranges are cut for ONE round of equally long
    // work-groups - the smallest range length L (in key tiles, at least two: a unit for each wave) for which
    // sum over (query, KV head) of ceil(tiles / L) fits the 256 CUs; a long sequence is cut into
    // more ranges than a short one.  Batches that do not fit one round even at the longest range a
    // work item may have run in several, longest items first.  Unused block tails of sequences that
    // alias table slots ride in the device block table and are masked by the kernel.
    if (bf16 && G <= 32 && p.total_S > 0 && ctx->forced_row_blocks == 0 &&
        (ctx->forced_attn_kernel == 0 || ctx->forced_attn_kernel == 3) &&
        std::all_of(p.suffix_len.begin(), p.suffix_len.end(), [](int32_t s) { return s <= 1; })) {
        constexpr int kCus = 256, kMinRange = 2;
        auto tiles_of_q = [&](int i) { return (p.prefix_len[i] + KT - 1) / KT; };
        auto items_at = [&](int L) {
            int64_t n = 0;
            for (int i = 0; i < p.B; ++i)
                if (p.suffix_len[i] > 0) n += (int64_t)c.n_kv_heads * std::max(1, (tiles_of_q(i) + L - 1) / L);
            return n;
        };
        int longest = 0;
        for (int i = 0; i < p.B; ++i)
            if (p.suffix_len[i] > 0) longest = std::max(longest, tiles_of_q(i));
        int L = kAttnMaxTiles;
        if (!ctx->compact && items_at(L) <= kCus) {                      // one round is possible: the shortest ranges that still fit it
            int lo = kMinRange, hi = kAttnMaxTiles;     // items_at is non-increasing in L
            while (lo < hi) {
                const int mid = (lo + hi) / 2;
                if (items_at(mid) <= kCus) hi = mid;
                else lo = mid + 1;
            }
            L = lo;
            // Up to 36 partials of a (query, KV head), 72 of four heads or fewer, are folded by the last work-group of it to end,
            // more by a launch of its own, which is 0.9 us.  Where the longest sequence would need that, ranges up to twice as
            // long - half of the work-groups stay, for the loads that they have in flight - are taken if they come out ahead: each
            // unit more that a wave takes is 0.65 us, each partial 0.035.  (One sequence, 28 / 4 heads, us a layer: 4.7 k tokens in 37
            // ranges of two tiles 9.9, in 25 of three 8.3; 15.7 k in 62 of four 12.8, in 31 of eight 12.3.)
            auto parts = [&](int l) { return (longest + l - 1) / l; };
            auto cost = [&](int l) { return 0.65 * ((l + 1) / 2) + 0.035 * parts(l) + (decode_folds(G, parts(l)) ? 0.0 : 0.9); };
            if (G <= 8 && !decode_folds(G, parts(lo)))
                for (int l = lo + 1; l <= std::min(lo * 2, kAttnMaxTiles); ++l)
                    if (cost(l) < cost(L) - 1e-9) L = l;
            // Up to six tiles - three units a wave - one range needs no partials and no arrival (one sequence of 200 tokens
            // 5.3 us against 7.0 in two ranges; of 500, eight tiles, 7.2 against 6.9 in four).
            if (longest <= 6) L = std::max(L, longest);
        }
        splits_of_q.assign(p.B, 1);
        p.max_splits = 1;
        for (int i = 0; i < p.B; ++i) {
            if (p.suffix_len[i] <= 0) continue;
            const int P = p.prefix_len[i];
            const int n_tiles = tiles_of_q(i);
            int ns = ctx->forced_splits > 0 ? ctx->forced_splits : (n_tiles + L - 1) / L;
            ns = std::max(ns, (n_tiles + kAttnMaxTiles - 1) / kAttnMaxTiles);
            ns = std::max(1, std::min(ns, std::max(n_tiles, 1)));
            splits_of_q[i] = ns;
            p.max_splits = std::max(p.max_splits, ns);
            if (ns > 1) p.n_part_slots += ns;
            const int32_t *bt = p.block_table.data() + (size_t)i * p.max_blocks;
            const uint8_t *pad_of = p.block_pad.empty() ? nullptr : p.block_pad.data() + (size_t)i * p.max_blocks;
            for (int h = 0; h < c.n_kv_heads; ++h)
                for (int s = 0; s < ns; ++s) {
                    AttnItem it{};
                    it.q = i; it.kvh = h; it.tile_begin = (int32_t)((int64_t)n_tiles * s / ns);
                    it.tile_end = (int32_t)((int64_t)n_tiles * (s + 1) / ns);
                    it.split = s; it.n_splits = ns; it.arrival = i * c.n_kv_heads + h; it.P = P; it.S = 1; it.cu = p.cu_seqlens[i];
                    it.append_bid = bt[P / kBlockTokens];
                    for (int k = 0; k < 16; ++k) {          // entries of the range's first units, clamped to the prefix
                        const int idx = std::min(it.tile_begin * (KT / kBlockTokens) + k, std::max((P + kBlockTokens - 1) / kBlockTokens - 1, 0));
                        it.bid[k] = bt[idx] | (pad_of ? (int32_t)((uint32_t)pad_of[idx] << kPadShift) : 0);
                    }
                    items.push_back(it);
                }
        }
        std::stable_sort(items.begin(), items.end(), [](const AttnItem &x, const AttnItem &y) {
            return x.tile_end - x.tile_begin > y.tile_end - y.tile_begin;
        });
        p.row_blocks = 1;
        p.n_items = (int32_t)items.size();
        p.pipelined = false;
        p.decode = true;
        p.fold = decode_folds(G, p.max_splits);
        if (p.max_splits > 1) place_partials(c, knobs, p, splits_of_q, items);
        p.n_arrivals = p.fold && p.max_splits > 1 ? p.B * c.n_kv_heads : 0;
        for (const AttnItem &it : items)
            if (it.tile_end - it.tile_begin > kAttnMaxTiles) return false;
        return true;
    }
    // key tiles of a query.  bf16 kernel: the tiles of the prefix (from the pool), then the tiles of
    // the suffix (from k_new / v_new); fp32 kernel: one paged sequence of P + S keys
    // the alternating-groups bf16 kernel, too, sees one sequence of P + S keys
    // It is chosen for launches of 14 us or more (estimated from the row tiles x key tiles of the batch at ~0.85 us
    // per 128 x 64 tile and CU) if its 256-row tiles are nearly as full as 128-row ones, of 80 us or more whatever
    // they are.  Measured: c3 (1140 items of ~24 tiles) 171 us against 226 us in the general kernel, c4 688 against 814 us in
    // the pipelined one.  The line is at 6 / 5, included, because five 128-row tiles that make three of 256 rows (40 / 8 heads,
    // 128 new tokens: the micro-batches of a cold cache) gain: 40 of those 1.085 times as fast as in the other kernels with
    // one partition count for all their queries, and another 1.1 .. 1.35 with plan_long's.
    // Shorter launches take it where plan_long puts it 20 % below the general and the pipelined kernel's model, 25 % where rows
    // are padded by more than that (of 160 batches of 4 .. 14 us those 32 are 1.08 .. 1.62 times as fast, 1.26 on average), and
    // from 15 % on where those leave the queries whole and this kernel does, too, or they have two of its row tiles each on average.
    // Of 84 batches between 15 and 20 % 28 are whole either way: 1.04 .. 1.57 times as fast, 1.27 on average; 20 are cut here alone and have the rows:
    // 0.96 .. 1.16, 1.07 on average (with fp16 partials 1.17); 11 have not: 0.93 .. 1.18 with fp16; 25 are cut by the others as well:
    // 0.89 .. 1.27, seven lose 2 .. 11 %.  What the short-launch kernel would take stays there, whose softmax weights, over eight
    // times as many key ranges, and partials lose less to rounding.
    //
    // The type of its partials (`wide`: fp32).  This kernel cuts queries that the others, or one partition count for the batch,
    // leave whole: those stay in fp32 to the end.  Where the batch's queries would be cut with fp16 partials in any case, they
    // are fp16 here as well: fp32 ones are twice the traffic (70 batches of 14 .. 300 us, 60 of 4 .. 14 us: 2.5 % slower on
    // average, 17 % at most, with fp32 in all of them).
    bool pp = false, wide = false;
    const bool any = p.total_S > 0, free_cut = any && !ctx->compact && ctx->forced_splits == 0;
    GeneralPlan general;
    BriefPlan brief;
    LongPlan lng;
    auto plan_others = [&] {
        general = plan_general(c, p, kAttnRows, KT, ctx->part_cap);
        if (ctx->short_rows > 0) brief = plan_brief(c, p, ctx->short_rows, KT, kAttnMaxTiles);
    };
    auto brief_wins = [&] { return brief.us < 0.85 * general.us; };      // (by more than the two models are unsure)
    if (bf16 && ctx->forced_row_blocks == 0) {
        if (ctx->forced_attn_kernel == 4) pp = true;
        else if (ctx->forced_attn_kernel == 0) {
            int64_t work = 0, work_pp = 0, n_q = 0;     // in 128-row tiles; the same with rows padded to this kernel's 256
            for (int i = 0; i < p.B; ++i)
                if (p.suffix_len[i] > 0) {
                    ++n_q;
                    const int64_t per_row_tile = (int64_t)c.n_kv_heads * (((int64_t)p.prefix_len[i] + p.suffix_len[i] + KT - 1) / KT);
                    work += per_row_tile * (((int64_t)p.suffix_len[i] * G + kAttnRows - 1) / kAttnRows);
                    work_pp += per_row_tile * 2 * (((int64_t)p.suffix_len[i] * G + 2 * kAttnRows - 1) / (2 * kAttnRows));
                }
            const double us = (double)work * 0.85 / 256.0;
            pp = us >= 80.0 || (!ctx->compact && us >= 14.0 && 5 * work_pp <= 6 * work);
            if (!pp && !ctx->compact && us >= 4.0 && us < 14.0) {
                plan_others();
                if (!brief_wins()) {
                    wide = free_cut && general.splits == 1;
                    lng = plan_long(c, p, 2 * kAttnRows, KT, ctx->part_cap, wide);
                    const bool sure = general.splits == 1 && (!lng.cut || (int64_t)p.total_S * G >= 4 * kAttnRows * n_q);
                    pp = lng.us < (5 * work_pp > 6 * work ? 0.75 : sure ? 0.85 : 0.8) * std::min(general.us, brief.us);
                }
            }
        }
        if (pp && free_cut && lng.range == 0) {
            wide = plan_general(c, p, 2 * kAttnRows, KT, ctx->part_cap, true).splits == 1;
            lng = plan_long(c, p, 2 * kAttnRows, KT, ctx->part_cap, wide);
        }
    }
    const bool unified = !bf16 || pp;
    p.pingpong = pp;
    p.part_f32 = pp && wide;
    auto tiles_of = [&](int P, int S) {
        return unified ? (P + S + KT - 1) / KT : (P + KT - 1) / KT + (S + KT - 1) / KT;
    };
    // bf16: 128 rows per work-group; 256 (two row blocks per wave, half the LDS traffic per flop but one
    // wave per SIMD) is kept as an option: it is slower until its matrix and vector work overlap
    const int rb = pp ? 2 : (bf16 && ctx->forced_row_blocks > 0) ? ctx->forced_row_blocks : 1;
    p.row_blocks = rb;
    int RT = bf16 ? kAttnRows * rb : kF32Rows;
    int want = 1, cut_range = 0;           // (cut_range: the length of a range in key tiles, where the queries are cut by that)
    if (ctx->forced_splits > 0) want = ctx->forced_splits;
    else if (ctx->compact) want = 1;
    else if (!bf16 && any) cut_range = plan_f32_range(c, p, RT, KT, ctx->part_cap);
    else if (pp && any) cut_range = lng.range;
    else if (any) {
        if (rb != 1) general = plan_general(c, p, RT, KT, ctx->part_cap);
        else if (general.us == GeneralPlan{}.us) plan_others();
        want = general.splits;
        // The short-launch kernel, where it is faster by more than the two models are unsure: of the batches that they
        // were fitted to it takes 451 of 740 and loses time in 8; over all 740 the call is 1.21 times as fast (1.24
        // if the faster kernel were known each time).  28 / 4 heads: one query of 1.1 k + 17 tokens 10.4 us against
        // 14.5; eight of 1 k + 17: 13 against 24; but one of 4.1 k + 128, whose rows fill 128-row tiles and
        // whose keys 32-row tiles would read four times as often, 25 against 22.
        if (ctx->forced_row_blocks == 0 && ctx->forced_attn_kernel == 0 && brief_wins()) {
            p.brief = true;
            cut_range = brief.range;
        }
    }
    if (bf16 && !pp && ctx->short_rows > 0 && ctx->forced_row_blocks == 0 && ctx->forced_attn_kernel == 5) {
        p.brief = true;
        if (ctx->forced_splits == 0 && !ctx->compact) cut_range = brief.range;
        want = std::max(1, ctx->forced_splits);
    }
    if (p.brief) {
        RT = ctx->short_rows;
    }
    splits_of_q.assign(p.B, 1);
    p.max_splits = 1;
    struct Bucket { int32_t first, count, tiles; };  // consecutive items of one (query, KV head, partition)
    // (a query has no more partitions than key tiles, whatever count a caller forces)
    auto partitions = [&](int n_tiles) {
        const int n = cut_range > 0 ? (n_tiles + cut_range - 1) / cut_range : want;
        return std::max(1, std::min(n, ctx->forced_splits > 0 ? n_tiles : n_tiles / 2));
    };
    int64_t n_flat = 0;
    for (int i = 0; i < p.B; ++i)
        if (p.suffix_len[i] > 0)
            n_flat += (int64_t)c.n_kv_heads * ((p.suffix_len[i] * G + RT - 1) / RT) * partitions(tiles_of(p.prefix_len[i], p.suffix_len[i]));
    std::vector<AttnItem> flat;
    std::vector<Bucket> buckets;
    flat.reserve((size_t)n_flat);
    int n_groups = 0;
    const bool by_row = !bf16 || p.brief;            // how this kernel keeps its partials
    for (int i = 0; i < p.B; ++i) {
        const int S = p.suffix_len[i], P = p.prefix_len[i];
        if (S <= 0) continue;
        const int n_tiles = tiles_of(P, S);
        // last block a tile load may touch: bf16 reads only prefix blocks from the pool
        const int last_blk = std::max(0, (unified ? (P + S + kBlockTokens - 1) / kBlockTokens
                                                  : (P + kBlockTokens - 1) / kBlockTokens) - 1);
        int ns = partitions(n_tiles);
        // block ids of a range fit LDS (the fp32 kernel can fetch those that do not from memory, which is slower)
        const int cap = !bf16 ? (ctx->compact ? n_tiles : kF32MaxTiles) : pp ? kPpMaxTiles : general_cap;
        if (ns < (n_tiles + cap - 1) / cap) { ns = (n_tiles + cap - 1) / cap; cap_bound = true; }
        ns = std::max(1, std::min(ns, n_tiles));
        const int n_mt = (S * G + RT - 1) / RT;
        // Partition boundaries.  A suffix tile of the bf16 kernel costs about 4 prefix tiles (its V
        // is transposed on the way into LDS), so the tiles are cut by weight, not by count - and a
        // cut by weight can leave a partition of prefix tiles longer than n_tiles / ns: where one
        // comes out longer than the block-id table allows, the query is cut into more.
        std::vector<int> cut;
        for (;; ++ns) {
            cut.assign(ns + 1, 0);
            const int npt = unified ? n_tiles : (P + KT - 1) / KT;
            const int w_new = p.brief ? 1 : 4;
            const int64_t total_w = npt + (int64_t)(n_tiles - npt) * w_new;
            int t = 0;
            int64_t acc = 0;
            for (int s = 1; s < ns; ++s) {
                const int64_t goal = total_w * s / ns;
                while (t < n_tiles - (ns - s) && acc + (t < npt ? 1 : w_new) <= goal) { acc += (t < npt ? 1 : w_new); ++t; }
                if (t < s) { acc += (t < npt ? 1 : w_new); ++t; }        // every partition gets a tile
                cut[s] = t;
            }
            cut[ns] = n_tiles;
            int longest = 0;
            for (int s = 0; s < ns; ++s) longest = std::max(longest, cut[s + 1] - cut[s]);
            if (longest <= cap || ns >= n_tiles) break;
            cap_bound = true;
        }
        splits_of_q[i] = ns;
        p.max_splits = std::max(p.max_splits, ns);
        if (by_row && ns > 1) p.n_part_slots += (int64_t)S * ns;
        const int32_t *bt = p.block_table.data() + (size_t)i * p.max_blocks;
        const uint8_t *pad_of = p.block_pad.empty() ? nullptr : p.block_pad.data() + (size_t)i * p.max_blocks;
        for (int h = 0; h < c.n_kv_heads; ++h) {
            for (int s = 0; s < ns; ++s) {
                const int t0 = cut[s], t1 = cut[s + 1];
                Bucket bucket{(int32_t)flat.size(), 0, t1 - t0};
                AttnItem proto{};                       // what the row tiles share
                proto.q = i; proto.kvh = h; proto.tile_begin = t0; proto.tile_end = t1; proto.split = s; proto.n_splits = ns;
                proto.P = P; proto.S = S; proto.cu = p.cu_seqlens[i];
                for (int k = 0; k < 16; ++k) {
                    const int idx = std::min(t0 * (KT / kBlockTokens) + k, last_blk);
                    proto.bid[k] = bt[idx] | (pad_of ? (int32_t)((uint32_t)pad_of[idx] << kPadShift) : 0);
                }
                if (pad_of && bf16 && !pp) {
                    const int n_fast = std::min(t1, P >> 6) - t0;
                    for (int k = t0 * 4; k < (t0 + std::max(n_fast, 0)) * 4; ++k) proto.n_pad_fast += pad_of[k];
                }
                for (int mt = 0; mt < n_mt; ++mt) {
                    flat.push_back(proto);
                    flat.back().m0 = mt * RT;
                    flat.back().arrival = n_groups + mt;
                    if (!by_row && ns > 1) flat.back().part0 = (int32_t)(p.n_part_slots + (int64_t)mt * ns);
                    ++bucket.count;
                    // (32-row tiles: eight, or four, of them share their keys' way into one L2, the next may go to
                    // another XCD, so that few (query, KV head) pairs still spread evenly)
                    if (bucket.count == (!bf16 ? 8 : p.brief ? 4 : INT32_MAX) && mt + 1 < n_mt) {
                        buckets.push_back(bucket);
                        bucket = Bucket{(int32_t)flat.size(), 0, t1 - t0};
                    }
                }
                buckets.push_back(bucket);
            }
            for (int mt = 0; mt < n_mt && !by_row; ++mt) groups.push_back(MergeGroup{h, mt * RT, ns, p.cu_seqlens[i], S, (int32_t)(p.n_part_slots + (int64_t)mt * ns), {0, 0}});
            n_groups += n_mt;
            if (!by_row && ns > 1) p.n_part_slots += (int64_t)n_mt * ns;
        }
    }
    p.n_groups = n_groups;
    // Longest buckets first, each to the XCD with the least work so far (key tiles x items): long
    // work-groups start early, XCDs finish together.
    std::stable_sort(buckets.begin(), buckets.end(), [](const Bucket &x, const Bucket &y) { return x.tiles > y.tiles; });
    std::vector<int32_t> xcd_of(buckets.size());
    int64_t xcd_load[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    int32_t xcd_items[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (size_t k = 0; k < buckets.size(); ++k) {
        int xcd = 0;
        for (int x = 1; x < 8; ++x)
            if (xcd_load[x] < xcd_load[xcd]) xcd = x;
        xcd_of[k] = xcd;
        xcd_load[xcd] += (int64_t)(buckets[k].tiles + 3) * buckets[k].count;
        xcd_items[xcd] += buckets[k].count;
    }
    const int32_t longest = *std::max_element(xcd_items, xcd_items + 8);
    AttnItem hole{};
    hole.q = -1; hole.n_splits = 1;
    items.assign((size_t)longest * 8, hole);
    int32_t at[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (size_t k = 0; k < buckets.size(); ++k)
        for (int32_t j = 0; j < buckets[k].count; ++j) {
            AttnItem &it = items[(size_t)at[xcd_of[k]]++ * 8 + xcd_of[k]];
            it = flat[buckets[k].first + j];
        }
    while (!items.empty() && items.back().q < 0) items.pop_back();
    p.n_items = (int32_t)items.size();
    // (the short-launch kernel: eight partials of a row in one round of loads; a launch of its own for them is 0.2 .. 1 us slower up
    // to there, and beyond, where one CU has a second round, 0.5 .. 5 us faster; the fp32 kernel: 0.3 .. 1.5 us slower up to eight
    // partials of 64 columns, beyond 0 .. 5 us faster, of 128 columns 0 .. 9 us faster from five on)
    // (inside the launch the partials of a row tile's tokens, up to 33, are addressed with 31 bits)
    p.fold = by_row && p.max_splits > 1 && (int64_t)33 * p.max_splits * c.n_q_heads * 512 <= INT32_MAX && (p.brief ? p.max_splits <= kShortFold : c.head_dim == 64 && !ctx->compact && p.max_splits <= kF32Fold);
    if (by_row && p.max_splits > 1) place_partials(c, knobs, p, splits_of_q, items);
    p.n_arrivals = p.fold ? n_groups : 0;
    // Which bf16 kernel (one row block per wave).  The pipelined one holds 132 KB of LDS, so one
    // work-group per CU: nothing hides a work-group's start-up and drain.  It wins when a launch is a
    // single round of work-groups or when they are long; many short ones (measured: 1140 work-groups
    // of ~20 key tiles, 743 vs 647 TFLOP/s) are better off two per CU in the general kernel.
    int64_t n_real = 0, fast_tiles = 0;
    for (const AttnItem &it : items)
        if (it.q >= 0) {
            ++n_real;
            fast_tiles += std::max(std::min(it.tile_end, it.P >> 6) - it.tile_begin, 0);
        }
    p.pipelined = bf16 && rb == 1 && !pp && !p.brief && n_real > 0 &&
                  (ctx->forced_attn_kernel == 1 || ctx->forced_attn_kernel == 2 ? ctx->forced_attn_kernel == 2
                                           : (n_real <= 2 * 256 || fast_tiles >= 48 * n_real));
    // every range's block ids must fit the table of the kernel that will run it
    const int limit = !bf16 ? (ctx->compact ? INT32_MAX : kF32MaxTiles) : pp ? kPpMaxTiles : p.pipelined ? kPipeMaxTiles : kAttnMaxTiles;
    p.longest_range = 0;
    for (const AttnItem &it : items)
        if (it.q >= 0) p.longest_range = std::max(p.longest_range, it.tile_end - it.tile_begin);
    return p.longest_range <= limit;
}

// Attention work list of the batch in `p`.  The general kernel keeps the block ids of at most
// kAttnMaxTiles key tiles per work item in LDS, the pipelined kernel (one work-group per CU, LDS to
// spare) kPipeMaxTiles: the batch is planned for the smaller table first; if that limit forced extra
// partitions and the pipelined kernel is the one chosen, it is planned again for the larger one
// (c4's 393-tile queries then run unsplit: no partials, no merge launch).
inline bool plan_attention(const tc_config &c, const PlanKnobs &knobs, Plan &p, std::vector<AttnItem> &items,
                           std::vector<int32_t> &splits_of_q, std::vector<MergeGroup> &groups)
{
    bool cap_bound = false;
    if (!plan_attention_pass(c, knobs, p, items, splits_of_q, groups, kAttnMaxTiles, cap_bound)) return false;
    if (cap_bound && p.pipelined && !p.pingpong && !p.decode) {
        PlanKnobs k2 = knobs;
        k2.forced_attn_kernel = 2;
        if (!plan_attention_pass(c, k2, p, items, splits_of_q, groups, kPipeMaxTiles, cap_bound)) return false;
    }
    return true;
}

inline bool parts_by_row(const tc_config &c, const Plan &p) { return (p.decode || c.dtype != TC_BF16 || p.brief) && p.max_splits > 1; }

inline int part_row_floats(const Plan &p) { return p.part_f32 ? 128 : 64; }      // a row's partial in fragment order, without its (maximum, sum)

// Does a launch of its own combine partials by row, and the table that it goes by (BatchDev::part_tab).
inline bool merges_rows(const tc_config &c, const Plan &p) { return parts_by_row(c, p) && !p.fold; }
inline size_t part_tab_ints(const Plan &p) { return (size_t)p.total_S + (p.part_stride == 0); }
inline void fill_part_tab(const Plan &p, const std::vector<int32_t> &splits_of_q, int32_t *out)
{
    int32_t at = 0;
    for (int i = 0; i < p.B; ++i) {
        const int32_t count = splits_of_q[i] > 1 ? splits_of_q[i] : 0;
        for (int n = p.cu_seqlens[i]; n < p.cu_seqlens[i + 1]; ++n, at += count) out[n] = p.part_stride ? count : at;
    }
    if (!p.part_stride) out[p.total_S] = at;
}

inline size_t part_floats(const tc_config &c, const Plan &p)      // all of the batch's partials, in floats
{
    if (parts_by_row(c, p)) return (size_t)p.n_part_slots * c.n_q_heads * (c.head_dim + 2);
    return (size_t)p.n_part_slots * p.row_blocks * kAttnRows * (part_row_floats(p) + 2);
}

// Where the parts of a plan stand in its device copy, in integers; only what the batch's kernels read
// is there (`n_*`: how many of each).
struct PlanLayout {
    size_t bt_row = 0;                     // integers per row of the block table
    size_t block_table, cu, prefix, suffix, tok_q, part_tab, items, groups;
    size_t seg_start, seg_len, seg_slot, stitch, rope_pos0, rope_freq;
    size_t total = 0;                      // a multiple of 8: the upload moves 16 bytes at a time
    // Arrival counters, behind what is uploaded and zeroed with it: 128 bytes each, as far apart as work items.  They are in the items
    // where the workspace of fixed size has no room for them, which is 0.1 .. 0.4 us a launch slower (arrive.h).
    size_t counters = 0, n_counter_ints = 0;
    bool lengths = false, tokens = false, merge_rows = false, merge_groups = false;
};
inline PlanLayout plan_layout(const tc_config &c, const Plan &p, size_t n_seg, size_t n_stitch, size_t n_items,
                              size_t n_groups)
{
    PlanLayout l;
    const size_t B = p.B;
    auto take = [&](size_t n) { const size_t o = l.total; l.total += (n + 7) & ~size_t(7); return o; };
    l.tokens = !p.decode && !p.pingpong && !p.brief;             // appended token by token, in extra work-groups
    l.lengths = l.tokens || n_stitch > 0;
    l.merge_rows = merges_rows(c, p);
    l.merge_groups = p.max_splits > 1 && !parts_by_row(c, p);
    // rows are padded to whole 16-byte chunks: the decode and short-launch kernels fetch them so, the long-launch
    // kernel where it can
    l.bt_row = p.compact && !p.decode && !p.brief ? (size_t)p.max_blocks : (size_t)(p.max_blocks + 3) & ~size_t(3);
    l.block_table = take(B * l.bt_row);
    l.prefix = take(l.lengths ? B : 0);
    l.cu = take(l.tokens ? B + 1 : 0); l.suffix = take(l.tokens ? B : 0); l.tok_q = take(l.tokens ? p.total_S : 0);
    l.seg_start = take(n_seg); l.seg_len = take(n_seg); l.seg_slot = take(n_seg);
    l.stitch = take(n_stitch * (sizeof(StitchBlk) / 4));
    l.part_tab = take(l.merge_rows ? part_tab_ints(p) : 0);
    l.items = take(n_items * (sizeof(AttnItem) / 4));
    l.groups = take(l.merge_groups ? n_groups * (sizeof(MergeGroup) / 4) : 0);
    l.rope_pos0 = take(p.rope ? B : 0); l.rope_freq = take(p.rope ? p.rope_rev_freq.size() * 2 : 0);
    l.total = std::max(l.total, size_t(8));
    l.counters = (l.total + 31) & ~size_t(31);
    l.n_counter_ints = (size_t)p.n_arrivals * (sizeof(AttnItem) / sizeof(int32_t));
    return l;
}

// The plan of a batch for a workspace of `max_ints` integers and `max_floats` floats of partials: the fastest
// one if it fits, else the one that takes the least space (which may still not fit: the caller looks).
inline bool plan_attention_within(const tc_config &c, const PlanKnobs &knobs, Plan &p, std::vector<AttnItem> &items,
                                  std::vector<int32_t> &splits_of_q, std::vector<MergeGroup> &groups, size_t max_ints,
                                  size_t max_floats)
{
    PlanKnobs k = knobs;
    k.part_cap = max_floats;
    if (!plan_attention(c, k, p, items, splits_of_q, groups)) return false;
    if (part_floats(c, p) <= max_floats &&
        plan_layout(c, p, 0, 0, items.size(), groups.size()).total <= max_ints) return true;
    k.compact = true;
    return plan_attention(c, k, p, items, splits_of_q, groups);
}

}  // namespace tc
