// Host-side compiler from a per-head plan to per-(batch, head, query tile) work records.
//
// Sec. 4.5 of the paper names the per-thread-block determination of the arrow pattern as
// the overhead that shows when little work remains.  Here the pattern is resolved once per
// distinct plan on the host, in integers: each record lists the key tiles a query tile has
// to visit (text tiles, then the tiles its rows' bands touch) and which of them are free of
// any masked pair, so the kernel never loads a fully masked tile and applies the element
// mask (Sec. 3.1: text quadrants whole, image-image band |i-j| <= w) only on edge tiles.
#include <stdint.h>

#include <algorithm>
#include <limits>
#include <new>
#include <vector>

#include "difa.h"
#include "difa_schedule.h"
#include "difa_testing.h"

namespace {

// Token order: the image tokens are [img0, img1), the text tokens the rest ([0, n_text) when the text
// comes first, [n_img, n_tokens) when the image does).  Key tiles are numbered in a rotated order that
// starts at the first tile holding a text key: position u is tile (u + rot) % n_kv_tiles.  With the
// text in front rot is 0; with the image in front the text tiles still come first in that order, so a
// record keeps the same two-range form.
struct Geometry {
    int n_text, n_tokens, bm, bn;
    int img0, img1;
    int rot, n_kv_tiles;
    int tile_at(int u) const { const int t = u + rot; return t >= n_kv_tiles ? t - n_kv_tiles : t; }
};

// Is there a pair (row in [i0,i1), key in [j0, j0+bn)) that must be masked out?
// w < 0 means a full head.  Keys >= n_tokens count as masked.
bool tile_needs_mask(const Geometry& g, int w, int i0, int i1, int j0) {
    const int j1 = j0 + g.bn;
    if (j1 > g.n_tokens) return true;
    if (w < 0) return false;
    const int qi0 = std::max(i0, g.img0), qi1 = std::min(i1, g.img1) - 1;  // image rows [qi0, qi1]
    const int kj0 = std::max(j0, g.img0), kj1 = std::min(j1, g.img1) - 1;  // image keys [kj0, kj1]
    if (qi0 > qi1 || kj0 > kj1) return false;
    return (kj1 - qi0 > w) || (qi1 - kj0 > w);
}

// Mask-free tiles of a range [begin, end) of positions in the rotated order: for the first range (prefix_only) the
// mask-free prefix, for the second the longest run of consecutive mask-free tiles.  Treating a mask-free tile as masked
// is always safe, so any sub-run is a valid answer.  A layer has thousands of records of hundreds of tiles, so the run
// comes from the band's edges and not from a look at every tile.
void mask_free_run(const Geometry& g, int w, int i0, int i1, int begin, int end, bool prefix_only,
                   int* run_begin, int* run_end) {
    *run_begin = *run_end = begin;
    if (begin >= end) return;
    const int qi0 = std::max(i0, g.img0), qi1 = std::min(i1, g.img1) - 1;          // image rows [qi0, qi1]
    if (w < 0 || qi0 > qi1) {
        // only the tile with the end of the sequence needs the mask
        const int tail = g.n_tokens % g.bn ? g.n_kv_tiles - 1 - g.rot : g.n_kv_tiles;   // its position
        if (tail < begin || tail >= end) *run_end = end;
        else if (prefix_only || tail - begin >= end - tail - 1) *run_end = tail;
        else { *run_begin = tail + 1; *run_end = end; }
        return;
    }
    if (prefix_only) {                                                             // the few tiles with text keys
        while (*run_end < end && !tile_needs_mask(g, w, i0, i1, g.tile_at(*run_end) * g.bn)) ++*run_end;
        return;
    }
    // The second range holds image keys only, tiles first, first + 1, ...: mask-free are those whose first key is at
    // most w below the last row, whose last key is at most w above the first row, and which lie inside the sequence.
    const int64_t first = g.tile_at(begin), low = std::max(0, qi1 - w), high = (int64_t)qi0 + w + 1;
    const int64_t t0 = (low + g.bn - 1) / g.bn, t1 = std::min<int64_t>(high, g.n_tokens) / g.bn;    // tiles [t0, t1)
    const int64_t b = std::max<int64_t>(begin, begin + (t0 - first)), e = std::min<int64_t>(end, begin + (t1 - first));
    if (b < e) { *run_begin = (int)b; *run_end = (int)e; }
}

}  // namespace

extern "C" int32_t difa_tile_shape(int32_t head_dim, int32_t dtype, int32_t* bm, int32_t* bn) {
    if ((head_dim != 64 && head_dim != 128) || (dtype != DIFA_DTYPE_BF16 && dtype != DIFA_DTYPE_F32))
        return 1;
    if (bm) *bm = 256;
    if (bn) *bn = 64;
    return 0;
}

namespace {
struct HeadSpan { size_t first, count; int64_t cost; };

// The records of a layer, head by head, query tiles in ascending order (`spans`, optional: where each head's lie).
// band_rows: query rows of the block-granular band's blocks, a multiple of the record's bm.
difa_status_t collect_records(int32_t band_rows, int32_t batch, int32_t heads, const int32_t* head_plan,
                              const int32_t* window, int32_t n_text, int32_t n_img, int32_t bm, int32_t bn, uint32_t flags,
                              std::vector<difa_work_item_t>& recs, std::vector<HeadSpan>* spans, int32_t* copy_heads,
                              int32_t* n_copy_out) {
    if (!head_plan || batch < 1 || heads < 1 || n_text < 0 || n_img < 0 ||
        bm < 1 || bn < 1 || band_rows < bm || band_rows % bm != 0 ||
        (flags & ~(uint32_t)(DIFA_FLAG_BLOCK_BAND | DIFA_FLAG_IMAGE_FIRST)) != 0)
        return DIFA_ERR_INVALID_ARG;
    const int64_t n64 = (int64_t)n_text + (int64_t)n_img;
    if (n64 < 1 || n64 > (int64_t)1 << 30) return DIFA_ERR_INVALID_ARG;
    for (int h = 0; h < heads; ++h) {
        const int mode = head_plan[h];
        if (mode != DIFA_HEAD_FULL && mode != DIFA_HEAD_ARROW && mode != DIFA_HEAD_CACHE && mode != DIFA_HEAD_ARROW_RESIDUAL)
            return DIFA_ERR_INVALID_ARG;
        if ((mode == DIFA_HEAD_ARROW || mode == DIFA_HEAD_ARROW_RESIDUAL) && (!window || window[h] < 0)) return DIFA_ERR_INVALID_ARG;
    }
    const bool image_first = (flags & DIFA_FLAG_IMAGE_FIRST) != 0 && n_text > 0 && n_img > 0;
    const bool block_band = (flags & DIFA_FLAG_BLOCK_BAND) != 0;
    const int n_kv_tiles = (int)((n64 + bn - 1) / bn);
    Geometry g{n_text, (int)n64, bm, bn, 0, 0, 0, n_kv_tiles};
    if (image_first) { g.img0 = 0; g.img1 = n_img; g.rot = n_img / bn; }
    else if (flags & DIFA_FLAG_IMAGE_FIRST) { g.img0 = 0; g.img1 = n_img; }      // one kind of token only
    else { g.img0 = n_text; g.img1 = g.n_tokens; }
    const int n_q_tiles = (g.n_tokens + bm - 1) / bm;
    // tiles that hold at least one text key: the first ones of the rotated order
    const int text_tiles = image_first ? n_kv_tiles - g.rot : (n_text + bn - 1) / bn;

    recs.clear();
    int n_copy = 0;
    for (int b = 0; b < batch; ++b) {
        for (int h = 0; h < heads; ++h) {
            const int mode = head_plan[h];
            if (mode == DIFA_HEAD_CACHE) {
                if (b == 0) {
                    if (copy_heads) copy_heads[n_copy] = h;
                    ++n_copy;
                }
                continue;
            }
            // A band that covers the whole image is full attention.
            const bool full = (mode == DIFA_HEAD_FULL) || (window[h] >= n_img - 1);
            const int w = full ? -1 : window[h];
            HeadSpan span{recs.size(), 0, 0};
            for (int qt = 0; qt < n_q_tiles; ++qt) {
                const int i0 = qt * bm, i1 = std::min(i0 + bm, g.n_tokens);
                // rows whose bands decide which key tiles are visited: the record's own, or with the block-granular
                // band those of the block of band_rows rows that holds the record
                const int v0 = block_band ? i0 / band_rows * band_rows : i0;
                const int v1 = block_band ? std::min(v0 + band_rows, g.n_tokens) : i1;
                difa_work_item_t r{};
                r.bh = b * heads + h;
                r.q_tile = qt;
                r.window = w;
                r.flags = mode == DIFA_HEAD_ARROW_RESIDUAL ? DIFA_ITEM_ADD_RESIDUAL : 0;   // arrow attention, then + r
                if (full && !image_first) {
                    r.kv0_end = n_kv_tiles;
                    r.kv1_begin = r.kv1_end = n_kv_tiles;
                } else if (full || v0 < g.img0 || v1 > g.img1) {
                    // every key: a full head, or a tile that holds text queries (they see every key).
                    // (Two ranges when the order is rotated, so that the sequence tail, the one tile a
                    // full head masks, ends the first range and the image tiles are mask-free as a run.)
                    r.kv0_end = text_tiles;
                    r.kv1_begin = text_tiles;
                    r.kv1_end = n_kv_tiles;
                } else {
                    r.kv0_end = text_tiles;
                    // image keys [lo, hi] that some row of the tile sees, as tiles; the tiles that also hold
                    // text keys are in the first range already
                    const int lo = std::max(g.img0, v0 - w);
                    const int hi = std::min(g.img1 - 1, (v1 - 1) + w);
                    if (image_first) {
                        const int t_lo = lo / bn, t_hi = std::min(hi / bn, g.rot - 1);
                        r.kv1_begin = text_tiles + t_lo;
                        r.kv1_end = std::max(r.kv1_begin, text_tiles + t_hi + 1);
                    } else {
                        r.kv1_begin = std::max(text_tiles, lo / bn);
                        r.kv1_end = std::max(r.kv1_begin, hi / bn + 1);
                    }
                }
                // Block-granular band (Sec. 3.3, Fig. 4): every visited block is dense, so the record is
                // masked like a full head's: on the sequence tail only.
                const int wm = block_band ? -1 : w;
                r.window = wm;
                int b0, e0;
                mask_free_run(g, wm, i0, i1, 0, r.kv0_end, true, &b0, &e0);
                r.nm0_end = e0;
                mask_free_run(g, wm, i0, i1, r.kv1_begin, r.kv1_end, false, &r.nm1_begin, &r.nm1_end);
                r.n_tiles = r.kv0_end + (r.kv1_end - r.kv1_begin);
                recs.push_back(r);
                span.cost += r.n_tiles;
            }
            span.count = recs.size() - span.first;
            if (spans) spans->push_back(span);
        }
    }
    *n_copy_out = n_copy;
    return DIFA_OK;
}

difa_status_t worklist_build(int32_t batch, int32_t heads, const int32_t* head_plan,
                             const int32_t* window, int32_t n_text, int32_t n_img,
                             int32_t bm, int32_t bn, int32_t n_xcd, uint32_t flags,
                             difa_work_item_t* items,
                             int32_t capacity, int32_t* n_items_out,
                             int32_t* copy_heads, int32_t* n_copy_out) {
    if (!n_items_out || n_xcd < 1 || n_xcd > 64 || capacity < 0 || (capacity > 0 && !items)) return DIFA_ERR_INVALID_ARG;
    std::vector<difa_work_item_t> recs;
    std::vector<HeadSpan> spans;
    int32_t n_copy = 0;
    const difa_status_t st = collect_records(bm, batch, heads, head_plan, window, n_text, n_img, bm, bn, flags, recs, &spans,
                                             copy_heads, &n_copy);
    if (st != DIFA_OK) return st;
    if (n_xcd == 1) {
        // Heaviest records first: the hardware hands workgroups out in index order, so the long
        // full-attention tiles start early and the short band tiles fill the tail.
        std::stable_sort(recs.begin(), recs.end(), [](const difa_work_item_t& a, const difa_work_item_t& b) {
            return a.n_tiles > b.n_tiles;
        });
    } else if (!recs.empty()) {
        // Workgroup p runs on accelerator die p % n_xcd, and every die has its own L2.  If the query
        // tiles of one head are spread over all dies, each die streams that head's K and V from
        // memory: n_xcd times the traffic.  So the records are laid out as n_xcd queues, queue x at
        // positions x, x + n_xcd, ...: heads in order of decreasing cost, the whole sequence cut into
        // n_xcd runs of equal cost, so that a head lives on one die (two where a cut falls inside it),
        // its query tiles run side by side and share the K/V tiles in that die's L2, and every die
        // gets the same amount of work.  Short queues are padded with records whose q_tile is -1.
        std::stable_sort(spans.begin(), spans.end(), [](const HeadSpan& a, const HeadSpan& b) { return a.cost > b.cost; });
        int64_t total = 0;
        for (const HeadSpan& sp : spans) total += sp.cost;
        std::vector<std::vector<difa_work_item_t>> queue((size_t)n_xcd);
        int64_t cum = 0;
        for (const HeadSpan& sp : spans)
            for (size_t k = 0; k < sp.count; ++k) {
                const difa_work_item_t& r = recs[sp.first + k];
                int64_t x = total > 0 ? ((2 * cum + r.n_tiles) * n_xcd) / (2 * total) : 0;
                x = std::min<int64_t>(std::max<int64_t>(x, 0), n_xcd - 1);
                queue[(size_t)x].push_back(r);
                cum += r.n_tiles;
            }
        // Inside a queue: longest records first (a query tile that holds text rows visits every key
        // tile and would otherwise start late and finish last), in classes of 16 key tiles so that
        // records of one head, which differ by a tile or two, stay next to each other.
        for (auto& q : queue)
            std::stable_sort(q.begin(), q.end(), [](const difa_work_item_t& a, const difa_work_item_t& b) {
                return a.n_tiles / 16 > b.n_tiles / 16;
            });
        size_t longest = 0;
        for (const auto& q : queue) longest = std::max(longest, q.size());
        difa_work_item_t pad{};
        pad.q_tile = -1;
        pad.window = -1;
        std::vector<difa_work_item_t> laid(longest * (size_t)n_xcd, pad);
        for (int x = 0; x < n_xcd; ++x)
            for (size_t k = 0; k < queue[(size_t)x].size(); ++k) laid[k * (size_t)n_xcd + (size_t)x] = queue[(size_t)x][k];
        while (!laid.empty() && laid.back().q_tile < 0) laid.pop_back();
        recs.swap(laid);
    }
    *n_items_out = (int32_t)recs.size();
    if (n_copy_out) *n_copy_out = n_copy;
    if ((int64_t)recs.size() > capacity) return capacity == 0 && !items ? DIFA_OK : DIFA_ERR_ALLOC;
    std::copy(recs.begin(), recs.end(), items);
    return DIFA_OK;
}
}  // namespace

extern "C" difa_status_t difa_worklist_build(int32_t batch, int32_t heads, const int32_t* head_plan,
                                             const int32_t* window, int32_t n_text, int32_t n_img,
                                             int32_t bm, int32_t bn, int32_t n_xcd, uint32_t flags,
                                             difa_work_item_t* items,
                                             int32_t capacity, int32_t* n_items_out,
                                             int32_t* copy_heads, int32_t* n_copy_out) {
    try {
        return worklist_build(batch, heads, head_plan, window, n_text, n_img, bm, bn, n_xcd, flags, items, capacity,
                              n_items_out, copy_heads, n_copy_out);
    } catch (const std::bad_alloc&) {
        return DIFA_ERR_ALLOC;
    }
}

difa_status_t difa::worklist_for_kernel(int32_t batch, int32_t heads, const int32_t* head_plan, const int32_t* window,
                                        int32_t n_text, int32_t n_img, int32_t rows, int32_t band_rows, int32_t bn,
                                        uint32_t flags, std::vector<difa_work_item_t>& recs, int32_t* copy_heads,
                                        int32_t* n_copy_out) {
    return collect_records(band_rows, batch, heads, head_plan, window, n_text, n_img, rows, bn, flags, recs, nullptr,
                           copy_heads, n_copy_out);
}

// ------------------------------------------------------------------------------------------
// Records -> per-workgroup segment lists for the persistent attention kernel.
//
// The hardware dispatcher would hand whole records to compute units as they free up; with records
// of a few hundred key tiles each, the last round leaves most of the chip idle (1584 equal records on
// 256 compute units: 6.19 rounds cost 7).  Here the distribution is computed on the host instead:
// whole records are dealt out, costliest first, to the least loaded workgroup of their die (which keeps
// the workgroups of a die on neighbouring query tiles of one head, marching through its K/V together),
// and the records that no longer fit under a target load are cut along their key-tile positions into
// pieces that fill the workgroups up to it.  A few targets above the mean load are tried.  A plan that its caller has not used lately is compiled while that
// caller waits, so the search works on loads and indices (a heap of the workgroups' loads, the part that
// every target has in common done once), and segments are written out for the plan that is kept only.
// ------------------------------------------------------------------------------------------
namespace {

// Cost model of a segment: difa::CostModel, in eighths of a plain key-tile iteration.
using difa::CostModel;
constexpr int kUnit = 8;                  // cost units per key-tile iteration
int piece_expected(const CostModel& m) { return m.piece + m.fold / 2; }   // what a piece is charged while cutting

// Masked tiles among positions [p0, p1) of a record's visiting order.
int masked_between(const difa_work_item_t& r, int p0, int p1) {
    int n = 0;
    const int e0 = std::min(p1, r.kv0_end);
    if (p0 < e0) n += std::max(0, e0 - std::max(p0, std::min(r.nm0_end, r.kv0_end)));
    const int b1 = std::max(p0, r.kv0_end);
    if (b1 < p1) {
        const int a = r.kv1_begin + (b1 - r.kv0_end), b = r.kv1_begin + (p1 - r.kv0_end);
        const int free = std::max(0, std::min(b, r.nm1_end) - std::max(a, r.nm1_begin));
        n += (b - a) - free;
    }
    return n;
}

int64_t tiles_cost(const CostModel& m, const difa_work_item_t& r, int p0, int p1) {
    return (int64_t)kUnit * (p1 - p0) + (int64_t)m.masked * masked_between(r, p0, p1);
}
int64_t whole_cost(const CostModel& m, const difa_work_item_t& r) { return tiles_cost(m, r, 0, r.n_tiles) + m.whole; }

// Positions of r from p0 on (at most `most`) whose iterations cost no more than `room` units.
int tiles_within(const CostModel& m, const difa_work_item_t& r, int p0, int most, int64_t room) {
    int lo = 0, hi = (int)std::min<int64_t>(most, room / kUnit);
    if (tiles_cost(m, r, p0, p0 + hi) <= room) return hi;
    while (hi - lo > 1) {
        const int mid = (lo + hi) / 2;
        if (tiles_cost(m, r, p0, p0 + mid) <= room) lo = mid; else hi = mid;
    }
    return lo;
}

difa_segment_t whole_segment(const difa_work_item_t& r) {
    difa_segment_t s{};
    s.bh = r.bh; s.q_tile = r.q_tile;
    s.kv0_end = r.kv0_end; s.nm0_end = r.nm0_end;
    s.kv1_begin = r.kv1_begin; s.kv1_end = r.kv1_end;
    s.nm1_begin = r.nm1_begin; s.nm1_end = r.nm1_end;
    s.window = r.window;
    s.flags = r.flags;
    s.pos_begin = 0; s.pos_end = r.n_tiles;
    s.part_slot = -1;
    s.merge_idx = -1;
    s.n_parts = 1;
    s.first_slot = -1;
    return s;
}

// Workgroups by load: a binary heap, the least loaded on top (the lower number among equals).
class LoadHeap {
public:
    void reset(int n) {
        at_.resize((size_t)n);
        for (int i = 0; i < n; ++i) at_[(size_t)i] = {0, i};
    }
    bool empty() const { return at_.empty(); }
    int top() const { return at_[0].second; }
    int64_t least() const { return at_[0].first; }
    void add_to_top(int64_t c) {
        std::pair<int64_t, int> x = at_[0];
        x.first += c;
        sink(x);
    }
    void pop() {
        const std::pair<int64_t, int> x = at_.back();
        at_.pop_back();
        if (!at_.empty()) sink(x);
    }
    int64_t most() const {
        int64_t m = 0;
        for (const auto& e : at_) m = std::max(m, e.first);
        return m;
    }

private:
    void sink(const std::pair<int64_t, int>& x) {       // x takes the place of the top
        const size_t n = at_.size();
        size_t i = 0;
        for (;;) {
            size_t k = 2 * i + 1;
            if (k >= n) break;
            if (k + 1 < n && at_[k + 1] < at_[k]) ++k;
            if (!(at_[k] < x)) break;
            at_[i] = at_[k];
            i = k;
        }
        at_[i] = x;
    }
    std::vector<std::pair<int64_t, int>> at_;
};

struct Placed { int wg, rec, pos_begin, pos_end; bool poured; };

// One die's share of the schedule.
struct DiePlan {
    std::vector<Placed> placed;        // in the order they were placed; the pieces of a record stand together
    int n_slots = 0;                   // pieces of cut records
    int64_t makespan = 0;
    int tried = 0;                     // how many times records were dealt out with cuts before this plan was settled on
};

// A die's records in order of decreasing cost, and the dealing of them.
struct Die {
    const CostModel& m;
    const std::vector<difa_work_item_t>& recs;
    const std::vector<std::pair<int64_t, int>>& order;     // (cost, index into recs)
    int64_t total;                                          // their cost
    int per_die, slot_budget;

    // Whole records only, each to the least loaded workgroup.
    void deal_whole(LoadHeap& heap, DiePlan& plan) const {
        heap.reset(per_die);
        plan.placed.clear();
        plan.n_slots = 0;
        for (const auto& o : order) {
            plan.placed.push_back({heap.top(), o.second, 0, recs[(size_t)o.second].n_tiles, false});
            heap.add_to_top(o.first);
        }
        plan.makespan = heap.most();
    }

    // A record goes whole to the least loaded workgroup (so neighbouring query tiles of a head run side by side and
    // share its K/V tiles in the die's L2) as long as that leaves the workgroup room for `spare` sixteenths more of
    // it; otherwise it is poured: laid into the room of the workgroup that is being filled, cut where that room ends,
    // the rest into the room of the workgroup that is then the least loaded, and so on.  With spare = 8 rooms are
    // of the order of a record when long records are cut (two or three pieces each, so the workgroup that folds them
    // together at the end reads one or two slots, not ten), and short records fill the gaps that remain.
    // [first, ...) are the records to deal; the heap and the plan hold what came before.  Returns false, with the plan
    // unfinished, when the records do not go in under the target.
    bool deal_and_pour(LoadHeap& heap, DiePlan& plan, size_t first, int64_t target, int spare) const {
        int cur = -1;                                                // the workgroup being filled, no longer in the heap
        int64_t cur_load = 0, most = 0;
        int64_t slack = target * per_die - total;                    // what closed rooms and cuts may waste
        for (size_t i = first; i < order.size(); ++i) {
            const int rec = order[i].second;
            const difa_work_item_t& r = recs[(size_t)rec];
            const int64_t c = order[i].first;
            if (!heap.empty() && heap.least() + c + c * spare / 16 <= target) {
                plan.placed.push_back({heap.top(), rec, 0, r.n_tiles, false});
                heap.add_to_top(c);
                continue;
            }
            const size_t piece_begin = plan.placed.size();
            int64_t dearest = 0;                                     // most loaded of the workgroups that take a piece
            int pos = 0;
            while (pos < r.n_tiles) {
                if (cur < 0 || target - cur_load - piece_expected(m) < (int64_t)kUnit * m.min_piece) {
                    // (the room left is too small for a piece; a short record may still fit whole)
                    if (cur >= 0 && pos == 0 && cur_load + c <= target) {
                        plan.placed.push_back({cur, rec, 0, r.n_tiles, true});
                        cur_load += c;
                        pos = r.n_tiles;
                        break;
                    }
                    if (cur >= 0) slack -= target - cur_load;
                    if (heap.empty() || slack < 0) return false;
                    most = std::max(most, cur_load);
                    cur = heap.top();
                    cur_load = heap.least();
                    heap.pop();
                }
                const int remaining = r.n_tiles - pos;
                const int64_t room = target - cur_load - piece_expected(m);
                const int64_t rest = tiles_cost(m, r, pos, r.n_tiles);
                int take = remaining;
                if (pos == 0 && cur_load + c <= target) {
                    // the whole record fits
                } else if (rest > room) {
                    if (plan.n_slots + (int)(plan.placed.size() - piece_begin) + 2 > slot_budget) return false;
                    take = room > 0 ? tiles_within(m, r, pos, remaining, room) : 0;
                    if (remaining - take < m.min_piece) take = remaining - m.min_piece;
                    if (take < m.min_piece) {                        // (room for less than a piece of masked tiles)
                        most = std::max(most, cur_load);
                        slack -= target - cur_load;
                        cur = -1;
                        continue;
                    }
                }
                plan.placed.push_back({cur, rec, pos, pos + take, true});
                cur_load += tiles_cost(m, r, pos, pos + take) + (take == r.n_tiles ? m.whole : piece_expected(m));
                dearest = std::max(dearest, cur_load);
                pos += take;
            }
            const int n = (int)(plan.placed.size() - piece_begin);
            if (n > 1) {
                plan.n_slots += n;
                slack -= (int64_t)n * piece_expected(m) - m.whole;
                // the pieces were charged half a fold each; with many pieces each one's share comes to more
                most = std::max(most, dearest + (int64_t)m.fold * (n - 1) / n - m.fold / 2);
            }
        }
        plan.makespan = std::max(std::max(most, cur_load), heap.most());
        return true;
    }

    // The best plan a few target loads give.
    DiePlan schedule() const {
        DiePlan best;
        int tried = 0;
        if (order.empty()) return best;
        LoadHeap heap;
        deal_whole(heap, best);
        // A die whose records are all too short to be cut (into two pieces of at least min_piece key tiles) has nothing to gain
        // below, and belongs to a layer whose call is over before a search would be: 24 heads of 64 and 333 tokens are compiled
        // in 13 us, in 140 with the search.
        const auto can_be_cut = [&](const std::pair<int64_t, int>& o) { return recs[(size_t)o.second].n_tiles >= 2 * m.min_piece; };
        int64_t uncut = 0;                                            // cost of the records that cannot be cut
        for (const auto& o : order) uncut += can_be_cut(o) ? 0 : o.first;
        if (uncut == total) return best;
        const int64_t mean = (total + per_die - 1) / per_die;
        DiePlan begun, plan;
        LoadHeap start;
        for (const int spare : {8, 0}) {
            if (best.makespan * 64 <= mean * 65) break;               // within 1.5 % of what no plan can beat
            // Every target from the mean load on deals the first records alike: as long as the least loaded
            // workgroup stays below the mean with the record and its spare room.
            start.reset(per_die);
            begun.placed.clear();
            size_t first = 0;
            while (first < order.size() && start.least() + order[first].first + order[first].first * spare / 16 <= mean) {
                begun.placed.push_back({start.top(), order[first].second, 0, recs[(size_t)order[first].second].n_tiles, false});
                start.add_to_top(order[first].first);
                ++first;
            }
            // Targets from just above the mean load up; the first one that holds everything is the plan.  How far up it
            // lies depends on how many cuts it takes: none of them costs more than `cut`, and a plan has about one for
            // every other workgroup.
            const int64_t cut = 2 * piece_expected(m) - m.whole;
            const auto holds_everything = [&](int64_t target) {
                // (every record longer than the target has to be cut)
                const int64_t longer = std::partition_point(order.begin(), order.end(), [&](const std::pair<int64_t, int>& o) {
                    return o.first > target; }) - order.begin();
                if (longer * cut > (target - mean) * per_die) return false;
                heap = start;
                plan.placed = begun.placed;
                plan.n_slots = 0;
                ++tried;
                return deal_and_pour(heap, plan, first, target, spare);
            };
            // Where most of the work is in records that cannot be cut, rooms end with a gap as a rule and no target may hold
            // everything: the two largest ones say so (not the largest alone: once in 500 layers a smaller one fits by luck).
            // With a record or two for each workgroup the whole search costs less than asking.
            if (order.size() > 2 * (size_t)per_die && 2 * uncut > total && mean + 3 * cut / 2 < best.makespan &&
                !holds_everything(mean + 3 * cut / 2) && !holds_everything(mean + cut))
                continue;
            for (const int64_t above : {cut / 8, cut / 3, 2 * cut / 3, cut, 3 * cut / 2}) {
                const int64_t target = mean + above;
                if (target >= best.makespan) break;
                if (!holds_everything(target)) continue;
                if (plan.makespan < best.makespan) std::swap(best, plan);
                break;
            }
            if (best.makespan * 100 <= mean * 104) break;
        }
        best.tried = tried;
        return best;
    }
};

difa_status_t schedule_build(const CostModel& m, const std::vector<difa_work_item_t>& recs, int32_t n_wg,
                             int32_t n_xcd, const double* die_speed, int64_t* die_span, difa_segment_t* segs,
                             int32_t seg_capacity, int32_t* wg_begin, int32_t* n_segs_out, difa_merge_item_t* merges,
                             int32_t merge_capacity, int32_t* n_merges_out, int32_t* n_slots_out, int32_t* tried = nullptr) {
    // heads in order of decreasing cost, the whole sequence cut into n_xcd runs whose costs are in
    // proportion to the dies' speeds (equal when none are given)
    std::vector<HeadSpan> spans;
    std::vector<int64_t> cost(recs.size());
    int64_t total = 0;
    for (size_t i = 0; i < recs.size();) {
        HeadSpan sp{i, 0, 0};
        for (; i < recs.size() && recs[i].bh == recs[sp.first].bh; ++i) sp.cost += cost[i] = whole_cost(m, recs[i]);
        sp.count = i - sp.first;
        total += sp.cost;
        spans.push_back(sp);
    }
    std::stable_sort(spans.begin(), spans.end(), [](const HeadSpan& a, const HeadSpan& b) { return a.cost > b.cost; });
    const int per_die = n_wg / n_xcd;
    const int slot_capacity = 2 * n_wg;
    std::vector<double> speed((size_t)n_xcd, 1.0);         // relative speeds of the dies (their clocks differ under load)
    if (die_speed)
        for (int x = 0; x < n_xcd; ++x) speed[(size_t)x] = die_speed[x] > 0.5 && die_speed[x] < 2.0 ? die_speed[x] : 1.0;
    std::vector<std::vector<std::pair<int64_t, int>>> die((size_t)n_xcd);
    std::vector<int64_t> die_cost((size_t)n_xcd);
    // The dies' plans for given shares of the work (up to a common factor), and the predicted finishing times of the first, the
    // last and all of them together, in cost units of a die of speed 1.  Given up with the first die that does not finish before `limit`.
    struct Plans {
        std::vector<DiePlan> die;
        double t_min = 0.0, t_max = 0.0, t_sum = 0.0;
    };
    const auto plans_for = [&](const std::vector<double>& share, double limit) {
        std::vector<double> upto((size_t)n_xcd + 1, 0.0);  // cumulative share of the work that dies 0 .. x-1 take
        {
            double sum = 0.0;
            for (int x = 0; x < n_xcd; ++x) sum += share[(size_t)x];
            for (int x = 0; x < n_xcd; ++x) upto[(size_t)x + 1] = upto[(size_t)x] + share[(size_t)x] / sum;
            upto[(size_t)n_xcd] = 2.0;
        }
        for (auto& d : die) d.clear();
        std::fill(die_cost.begin(), die_cost.end(), 0);
        int64_t cum = 0;
        int x_at = 0;
        for (const HeadSpan& sp : spans)
            for (size_t k = sp.first; k < sp.first + sp.count; ++k) {
                const double mid = total > 0 ? (double)(2 * cum + cost[k]) / (double)(2 * total) : 0.0;
                while (x_at < n_xcd - 1 && mid >= upto[(size_t)x_at + 1]) ++x_at;
                die[(size_t)x_at].push_back({cost[k], (int)k});
                die_cost[(size_t)x_at] += cost[k];
                cum += cost[k];
            }
        Plans p;
        p.die.resize((size_t)n_xcd);
        int slots_so_far = 0;
        for (int x = 0; x < n_xcd; ++x) {
            // costliest records first (a query tile that holds text rows visits every key tile); the interior
            // query tiles of a head cost the same and stay neighbours
            std::stable_sort(die[(size_t)x].begin(), die[(size_t)x].end(),
                             [](const std::pair<int64_t, int>& a, const std::pair<int64_t, int>& b) { return a.first > b.first; });
            const int budget = slot_capacity - slots_so_far - 2 * per_die * (n_xcd - 1 - x);   // this die's share of the slots
            p.die[(size_t)x] = Die{m, recs, die[(size_t)x], die_cost[(size_t)x], per_die, budget}.schedule();
            slots_so_far += p.die[(size_t)x].n_slots;
            if (tried) *tried += p.die[(size_t)x].tried;
            const double t = (double)p.die[(size_t)x].makespan / speed[(size_t)x];
            p.t_min = x == 0 ? t : std::min(p.t_min, t);
            p.t_max = std::max(p.t_max, t);
            p.t_sum += t;
            if (t >= limit) break;
        }
        return p;
    };
    const auto apart = [&](const Plans& p) { return p.t_min > 0.0 && (p.t_max - p.t_min) * n_xcd > 0.03 * p.t_sum; };
    // First the work is handed out in proportion to the dies' speeds; where the plans that come out of it would finish more
    // than three hundredths apart (a die whose records had to be cut carries the overhead of the cuts), the shares are corrected
    // by that and the plans made again, and kept if they are better.
    // Where the last die is still predicted to end well behind the mean, equal shares are tried as well, and corrected where they are
    // earlier.  A layer with no more records than workgroups needs them most: there a share a few hundredths larger can be one record
    // more than the die has workgroups, which takes as long as two, or has records cut to avoid that. (512 records of 1024 keys at
    // head_dim 128, one for each workgroup: 39 us, and 51 in those processes whose measured die speeds gave some die 65 of them; 4096
    // keys: 122 us, 131-142 with records cut; head_dim 64 72.7 and 80.)  They come after the correction, not in its place: that way some
    // layers ended up to three times as late (6 heads, 3658 tokens).  First calls wait for all this, hence the limit: 139 us in
    // the mean for such a layer on uneven dies, 132 with the correction alone.
    Plans best = plans_for(speed, std::numeric_limits<double>::infinity());
    const auto try_shares = [&](const std::vector<double>& share) {
        Plans next = plans_for(share, best.t_max);
        if (next.t_max >= best.t_max) return false;
        best = std::move(next);
        return true;
    };
    const auto try_corrected = [&](std::vector<double> share) {      // (the shares that `best` was made for)
        for (int x = 0; x < n_xcd; ++x)
            share[(size_t)x] *= (best.t_sum / n_xcd) / ((double)best.die[(size_t)x].makespan / speed[(size_t)x]);
        try_shares(share);
    };
    const auto late = [&](double by) { return best.t_max * n_xcd > (1.0 + by) * best.t_sum; };   // the last die, behind the mean
    const bool uneven = *std::max_element(speed.begin(), speed.end()) > *std::min_element(speed.begin(), speed.end());
    if (apart(best)) try_corrected(speed);
    if (uneven && late(recs.size() <= (size_t)n_wg ? 0.02 : 0.1)) {
        const std::vector<double> equal((size_t)n_xcd, 1.0);
        if (try_shares(equal) && apart(best) && late(0.1)) try_corrected(equal);
    }
    std::vector<DiePlan>& plans = best.die;

    // ---- the plans written out: segments grouped by workgroup (workgroup w of die x is number w * n_xcd + x)
    int64_t n_segs = 0, n_slots = 0, n_merges = 0;
    for (const DiePlan& p : plans) {
        n_segs += (int64_t)p.placed.size();
        n_slots += p.n_slots;
        for (size_t i = 0; i < p.placed.size(); ++i)
            n_merges += p.placed[i].pos_begin == 0 && p.placed[i].pos_end < recs[(size_t)p.placed[i].rec].n_tiles;
    }
    *n_segs_out = (int32_t)n_segs;
    *n_merges_out = (int32_t)n_merges;
    *n_slots_out = (int32_t)n_slots;
    if (n_segs > seg_capacity || n_merges > merge_capacity) return DIFA_ERR_ALLOC;
    std::fill(wg_begin, wg_begin + n_wg + 1, 0);
    for (int x = 0; x < n_xcd; ++x) {
        if (die_span) die_span[x] = plans[(size_t)x].makespan;
        for (const Placed& pl : plans[(size_t)x].placed) ++wg_begin[pl.wg * n_xcd + x + 1];
    }
    for (int w = 0; w < n_wg; ++w) wg_begin[w + 1] += wg_begin[w];
    std::vector<int32_t> at(wg_begin, wg_begin + n_wg);              // next free place of each workgroup
    std::vector<int32_t> poured_from((size_t)n_wg, -1);              // where its poured segments begin
    int32_t slot = 0, merge = 0;
    for (int x = 0; x < n_xcd; ++x) {
        const std::vector<Placed>& placed = plans[(size_t)x].placed;
        for (size_t i = 0; i < placed.size();) {
            size_t j = i + 1;                                        // placed[i, j): one record
            const difa_work_item_t& r = recs[(size_t)placed[i].rec];
            while (j < placed.size() && placed[j].rec == placed[i].rec) ++j;
            const int n = (int)(j - i), first_slot = slot;
            for (; i < j; ++i) {
                const int w = placed[i].wg * n_xcd + x;
                if (placed[i].poured && poured_from[(size_t)w] < 0) poured_from[(size_t)w] = at[(size_t)w];
                difa_segment_t& s = segs[at[(size_t)w]++];
                s = whole_segment(r);
                s.pos_begin = placed[i].pos_begin;
                s.pos_end = placed[i].pos_end;
                if (n > 1) {
                    s.first_slot = first_slot;
                    s.part_slot = slot++;
                    s.merge_idx = merge;
                    s.n_parts = n;
                }
            }
            if (n > 1) merges[merge++] = difa_merge_item_t{r.bh, r.q_tile, first_slot, n};
        }
    }
    // A poured room holds the tail of one record and the head of the next one, neighbouring query tiles of
    // one head as a rule.  Run in the order of their first key position (the shorter one first among equals),
    // the workgroups of the die walk through that head's K/V within a fraction of a record of each other and
    // share the tiles in the die's L2, as they do on whole records; the pieces of a record may finish in any
    // order, since the last one to arrive folds them.
    for (int w = 0; w < n_wg; ++w)
        if (poured_from[(size_t)w] >= 0)
            std::stable_sort(segs + poured_from[(size_t)w], segs + wg_begin[w + 1], [](const difa_segment_t& a, const difa_segment_t& b) {
                return a.pos_begin != b.pos_begin ? a.pos_begin < b.pos_begin
                                                  : a.pos_end - a.pos_begin < b.pos_end - b.pos_begin;
            });
    return DIFA_OK;
}
}  // namespace

extern "C" difa_status_t difa_schedule_build(const difa_work_item_t* items, int32_t n_items, int32_t n_wg,
                                             int32_t n_xcd, difa_segment_t* segs, int32_t seg_capacity,
                                             int32_t* wg_begin, int32_t* n_segs_out, difa_merge_item_t* merges,
                                             int32_t merge_capacity, int32_t* n_merges_out, int32_t* n_slots_out) {
    if (n_items < 0 || (n_items > 0 && !items) || n_wg < 1 || n_xcd < 1 || n_wg % n_xcd != 0 || !wg_begin ||
        !n_segs_out || !n_merges_out || !n_slots_out || seg_capacity < 0 || merge_capacity < 0 ||
        (seg_capacity > 0 && !segs) || (merge_capacity > 0 && !merges))
        return DIFA_ERR_INVALID_ARG;
    try {
        std::vector<difa_work_item_t> recs;
        for (int32_t i = 0; i < n_items; ++i) {
            if (items[i].q_tile < 0) continue;
            if (items[i].n_tiles < 1) return DIFA_ERR_INVALID_ARG;
            recs.push_back(items[i]);
        }
        std::stable_sort(recs.begin(), recs.end(), [](const difa_work_item_t& a, const difa_work_item_t& b) {
            return a.bh != b.bh ? a.bh < b.bh : a.q_tile < b.q_tile;
        });
        return schedule_build(difa::kGenericCosts, recs, n_wg, n_xcd, nullptr, nullptr, segs, seg_capacity, wg_begin, n_segs_out,
                              merges, merge_capacity, n_merges_out, n_slots_out);
    } catch (const std::bad_alloc&) {
        return DIFA_ERR_ALLOC;
    }
}

difa_status_t difa::schedule_for_dies(const CostModel& m, const std::vector<difa_work_item_t>& recs, int32_t n_wg, int32_t n_xcd,
                                      const double* die_speed, int64_t* die_span, difa_segment_t* segs,
                                      int32_t seg_capacity, int32_t* wg_begin, int32_t* n_segs_out,
                                      difa_merge_item_t* merges, int32_t merge_capacity, int32_t* n_merges_out,
                                      int32_t* n_slots_out) {
    return schedule_build(m, recs, n_wg, n_xcd, die_speed, die_span, segs, seg_capacity, wg_begin, n_segs_out,
                          merges, merge_capacity, n_merges_out, n_slots_out);
}

// ---- views for the library's tests (difa_testing.h)
extern "C" difa_status_t difa_testing_records(int32_t batch, int32_t heads, const int32_t* head_plan, const int32_t* window,
                                              int32_t n_text, int32_t n_img, int32_t rows, int32_t head_dim, uint32_t flags,
                                              difa_work_item_t* items, int32_t capacity, int32_t* n_items) {
    int32_t band_rows = 0, bn = 0, n_copy = 0;
    if (!n_items || difa_tile_shape(head_dim, DIFA_DTYPE_BF16, &band_rows, &bn) != 0) return DIFA_ERR_INVALID_ARG;
    try {
        std::vector<difa_work_item_t> recs;
        const difa_status_t st = difa::worklist_for_kernel(batch, heads, head_plan, window, n_text, n_img, rows, band_rows, bn, flags,
                                                           recs, nullptr, &n_copy);
        if (st != DIFA_OK) return st;
        *n_items = (int32_t)recs.size();
        if ((int64_t)recs.size() > capacity) return capacity == 0 && !items ? DIFA_OK : DIFA_ERR_ALLOC;
        std::copy(recs.begin(), recs.end(), items);
        return DIFA_OK;
    } catch (const std::bad_alloc&) {
        return DIFA_ERR_ALLOC;
    }
}

extern "C" difa_status_t difa_testing_schedule(const difa_work_item_t* items, int32_t n_items, int32_t head_dim, int32_t n_wg,
                                               int32_t n_xcd, const double* die_speed, int64_t* die_span, difa_segment_t* segs,
                                               int32_t seg_capacity, int32_t* wg_begin, int32_t* n_segs, difa_merge_item_t* merges,
                                               int32_t merge_capacity, int32_t* n_merges, int32_t* n_slots, int32_t* tried) {
    *tried = 0;
    try {
        const std::vector<difa_work_item_t> recs(items, items + n_items);
        return schedule_build(difa::kernel_costs(head_dim), recs, n_wg, n_xcd, die_speed, die_span, segs, seg_capacity, wg_begin,
                              n_segs, merges, merge_capacity, n_merges, n_slots, tried);
    } catch (const std::bad_alloc&) {
        return DIFA_ERR_ALLOC;
    }
}
