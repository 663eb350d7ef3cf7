// Host-side integer work of the packed variable-length attention library:
// first-fit packing, per-bin layout, tile shapes, per-tile work lists and the
// per-head E4M3 quantiser.  Pure host code; nothing here touches the GPU.
//
// Paper: section 2.2.1 (2) "Data Packing" (samples are concatenated into
// sequences close to the maximum context length, no padding tokens) and
// section 2.2.1 (1) (compute on valid tokens only).  The paper names no bin
// rule; online first-fit in arrival order is this library's reading.
#include "common.h"

#include <algorithm>
#include <cmath>
#include <cstring>
#include <vector>

namespace va {

thread_local char g_error[512] = "";

int fail(int code, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_error, sizeof(g_error), fmt, ap);
    va_end(ap);
    return code;
}

// Heads of one KV group that a forward / dQ workgroup stacks on its 128 rows.
int heads_per_block(int32_t Hq, int32_t Hkv) {
    const int G = Hq / Hkv;
    int hpb = 1;
    while (hpb * 2 <= 8 && G % (hpb * 2) == 0) hpb *= 2;
    return hpb;
}

int tile_shape(int32_t pass, int32_t D, int32_t Hq, int32_t Hkv, int32_t* rows, int32_t* cols) {
    if (!head_dim_supported(D)) return fail(VA_EUNSUPPORTED, "head_dim %d not in {48,64,80,96,128,160,192,256}", D);
    if (Hq <= 0 || Hkv <= 0 || Hq % Hkv != 0)
        return fail(VA_EUNSUPPORTED, "num_q_heads %d is not a positive multiple of num_kv_heads %d", Hq, Hkv);
    switch (pass) {
        case VA_PASS_FWD:
            *rows = kFwdBlockRows / heads_per_block(Hq, Hkv);
            *cols = kFwdKvTile;
            return VA_OK;
        case VA_PASS_BWD_DQ:
            *rows = kDqBlockRows / heads_per_block(Hq, Hkv);
            *cols = kDqKvTile;
            return VA_OK;
        case VA_PASS_BWD_DKDV:
            *rows = kDkdvKvRows;
            *cols = dkdv_q_tile(D);
            return VA_OK;
        default:
            return fail(VA_EUNSUPPORTED, "unknown pass %d", pass);
    }
}

int works_per_item(int32_t pass, int32_t Hq, int32_t Hkv) {
    if (pass == VA_PASS_BWD_DKDV) return Hkv;
    return Hkv * ((Hq / Hkv) / heads_per_block(Hq, Hkv));
}

WorklistLayout worklist_layout(int32_t pass, int32_t D, int32_t Hq, int32_t Hkv, int32_t num_items, int32_t num_merges) {
    WorklistLayout l;
    l.num_workgroups = persistent_workgroups(pass, D);
    l.works_per_item = works_per_item(pass, Hq, Hkv);
    l.num_works = num_items * l.works_per_item;
    l.num_items = num_items;
    l.item_rec = 2;
    l.table_rec = l.item_rec + num_items;
    l.id_rec = l.table_rec + l.num_workgroups * (kTableWordsPerWorkgroup / 8);
    l.num_merges = num_merges;
    l.flags = 0;
    l.few = false;
    l.few_splits = 1;
    l.merge_rec = l.id_rec + (l.num_works + 7) / 8;
    l.total_recs = l.merge_rec + num_merges;
    return l;
}

}  // namespace va

using namespace va;

namespace {

struct Keyed {
    int32_t work;    // inner-loop steps of the item per head (the order of the list)
    int32_t sample;  // index of its sample
    WorkItem it;
};

// Heaviest first, ties in the order given: a counting sort where the step counts are small numbers, as they are
// for every stream but a few items of enormous samples.
void sort_heaviest_first(std::vector<Keyed>& items) {
    int32_t top = 0;
    for (const Keyed& k : items) top = std::max(top, k.work);
    if ((size_t)top > 4 * items.size() + 1024) {
        std::stable_sort(items.begin(), items.end(), [](const Keyed& a, const Keyed& b) { return a.work > b.work; });
        return;
    }
    std::vector<int32_t> at((size_t)top + 2, 0);  // at[top - work + 1] counts, then at[top - work] is the next place
    for (const Keyed& k : items) ++at[(size_t)(top - k.work) + 1];
    for (size_t i = 1; i < at.size(); ++i) at[i] += at[i - 1];
    std::vector<Keyed> sorted(items.size());
    for (const Keyed& k : items) sorted[(size_t)at[(size_t)(top - k.work)]++] = k;
    items.swap(sorted);
}

// Least-loaded-first queue of workgroups (ties: lowest index): a binary heap of (load, index) in one word each,
// in which the workgroup at the top takes the next work and sinks to its new place.
class LeastLoaded {
public:
    // workgroups first, first + step, ... below end, all idle
    LeastLoaded(int32_t first, int32_t end, int32_t step) {
        for (int32_t w = first; w < end; w += step) heap_.push_back((uint64_t)w);  // equal loads, ascending: a heap
    }
    // gives the least-loaded workgroup a work of this cost: returns its index
    int32_t give(int64_t cost) {
        const uint64_t key = heap_[0] + ((uint64_t)cost << kIndexBits);
        const int32_t who = (int32_t)(key & ((1u << kIndexBits) - 1));
        last_finish_ = std::max(last_finish_, (int64_t)(key >> kIndexBits));
        const size_t n = heap_.size();
        size_t i = 0;
        for (;;) {
            size_t c = 2 * i + 1;
            if (c >= n) break;
            if (c + 1 < n && heap_[c + 1] < heap_[c]) ++c;
            if (heap_[c] >= key) break;
            heap_[i] = heap_[c];
            i = c;
        }
        heap_[i] = key;
        return who;
    }
    int64_t last_finish() const { return last_finish_; }  // largest load so far

private:
    static constexpr int kIndexBits = 16;  // workgroups of a launch stay far below 2^16, loads below 2^48
    std::vector<uint64_t> heap_;
    int64_t last_finish_ = 0;
};

// dK/dV pass: one workgroup runs one work, and the hardware hands the works to free workgroup slots in list
// order (heaviest first).  With few heavy works per slot the last round can leave most slots idle (257 equal
// works on 256 slots take two rounds).  This routine replays that dispatch on `slots` slots and, while the
// work that finishes last ends later than 1.04 times the lower bound max(mean load, heaviest work) (and, to
// begin with, later than 1.1 times), cuts the query tiles of its key tile into pieces of about an eighth of
// the lower bound each.  A piece is an item of its own with a partial-sum slot; `merges` receives one record
// per split tile.  At most max_slots pieces in all.
void split_late_tiles(std::vector<Keyed>& items, std::vector<WorkItem>& merges, int32_t G, int32_t Hkv,
                      int32_t slots, int32_t max_slots) {
    auto cost = [&](const Keyed& k) { return (int64_t)k.work * G + kWorkFixedCost; };
    int32_t used = 0;
    for (int32_t round = 0; round < max_slots; ++round) {
        sort_heaviest_first(items);
        int64_t total = 0, heaviest = 0, last_finish = 0;
        int32_t last_item = -1;
        LeastLoaded queue(0, slots, 1);
        for (size_t i = 0; i < items.size(); ++i) {
            const int64_t c = cost(items[i]);
            for (int32_t g = 0; g < Hkv; ++g) queue.give(c);
            total += c * Hkv;
            heaviest = std::max(heaviest, c);
            if (queue.last_finish() > last_finish) {
                last_finish = queue.last_finish();
                last_item = (int32_t)i;
            }
        }
        if (last_item < 0) return;
        const int64_t bound = std::max((total + slots - 1) / slots, heaviest);
        if (last_finish * 100 <= bound * (used == 0 ? 110 : 104)) return;
        Keyed& k = items[(size_t)last_item];
        if (dkdv_item_slot(k.it.w[1]) >= 0) return;  // a piece is not split again
        const int32_t n = k.it.w[4];                  // query tiles of the item
        const int32_t per = (int32_t)std::max<int64_t>(1, bound / 8 / G);
        const int32_t pieces = std::min({(n + per - 1) / per, kMaxPiecesPerTile, max_slots - used});
        if (pieces < 2) return;
        const Keyed whole = k;
        merges.push_back({{whole.it.w[0], whole.it.w[1], used, pieces, whole.it.w[3], whole.it.w[4], 0, 0}});
        int32_t at = whole.it.w[3];
        for (int32_t j = 0; j < pieces; ++j) {
            const int32_t count = n / pieces + (j < n % pieces ? 1 : 0);
            Keyed piece = whole;
            piece.work = count;
            piece.it.w[1] = whole.it.w[1] | (used + j + 1) << 8;
            piece.it.w[3] = at;
            piece.it.w[4] = count;
            at += count;
            if (j == 0) items[(size_t)last_item] = piece;
            else items.push_back(piece);
        }
        used += pieces;
    }
}

}  // namespace

extern "C" {

const char* va_last_error(void) { return g_error; }

int va_pack_first_fit(const int32_t* lens, int32_t N, int32_t budget,
                      int32_t* bin_of_sample, int32_t* pos_in_bin, int32_t* num_bins) {
    if (N < 0 || budget < 0 || !num_bins || (N > 0 && (!lens || !bin_of_sample || !pos_in_bin)))
        return fail(VA_EINVAL, "va_pack_first_fit: null pointer or negative size");
    for (int32_t i = 0; i < N; ++i) {
        if (lens[i] < 0) return fail(VA_EINVAL, "va_pack_first_fit: lens[%d] = %d is negative", i, lens[i]);
        if (lens[i] > budget)
            return fail(VA_ESIZE, "va_pack_first_fit: lens[%d] = %d exceeds the budget %d", i, lens[i], budget);
    }
    std::vector<int32_t> free_tokens, count;
    for (int32_t i = 0; i < N; ++i) {
        size_t b = 0;
        while (b < free_tokens.size() && free_tokens[b] < lens[i]) ++b;
        if (b == free_tokens.size()) {
            free_tokens.push_back(budget);
            count.push_back(0);
        }
        free_tokens[b] -= lens[i];
        bin_of_sample[i] = (int32_t)b;
        pos_in_bin[i] = count[b]++;
    }
    *num_bins = (int32_t)free_tokens.size();
    return VA_OK;
}

int va_bin_layout(const int32_t* lens, const int32_t* prefix, int32_t n,
                  int32_t* cu_seqlens, int32_t* prefix_lens, int32_t* max_seqlen) {
    if (n < 0 || !cu_seqlens || !max_seqlen || (n > 0 && !lens) || (prefix && !prefix_lens))
        return fail(VA_EINVAL, "va_bin_layout: null pointer or negative size");
    int64_t sum = 0;
    int32_t mx = 0;
    for (int32_t s = 0; s < n; ++s) {
        if (lens[s] < 0) return fail(VA_EINVAL, "va_bin_layout: lens[%d] is negative", s);
        if (prefix && (prefix[s] < 0 || prefix[s] > lens[s]))
            return fail(VA_EINVAL, "va_bin_layout: prefix[%d] = %d outside [0, %d]", s, prefix[s], lens[s]);
        sum += lens[s];
        if (sum > INT32_MAX) return fail(VA_ESIZE, "va_bin_layout: more than 2^31-1 tokens");
        mx = std::max(mx, lens[s]);
    }
    cu_seqlens[0] = 0;
    for (int32_t s = 0; s < n; ++s) {
        cu_seqlens[s + 1] = cu_seqlens[s] + lens[s];
        if (prefix) prefix_lens[s] = prefix[s];
    }
    *max_seqlen = mx;
    return VA_OK;
}

int va_tile_shape(int32_t pass, int32_t head_dim, int32_t num_q_heads, int32_t num_kv_heads,
                  int32_t* rows, int32_t* cols) {
    if (!rows || !cols) return fail(VA_EINVAL, "va_tile_shape: null pointer");
    return tile_shape(pass, head_dim, num_q_heads, num_kv_heads, rows, cols);
}

static int check_cu(const int32_t* cu, int32_t n, const char* who) {
    if (n < 0 || !cu) return fail(VA_EINVAL, "%s: null cu_seqlens or negative num_seqs", who);
    if (cu[0] != 0) return fail(VA_EINVAL, "%s: cu_seqlens[0] = %d, expected 0", who, cu[0]);
    for (int32_t s = 0; s < n; ++s)
        if (cu[s + 1] < cu[s]) return fail(VA_EINVAL, "%s: cu_seqlens decreases at %d", who, s);
    return VA_OK;
}

int va_worklist_size(const int32_t* cu, int32_t n, int32_t pass, int32_t D,
                      int32_t Hq, int32_t Hkv, size_t* bytes) {
    if (!bytes) return fail(VA_EINVAL, "va_worklist_size: null pointer");
    int rc = check_cu(cu, n, "va_worklist_size");
    if (rc) return rc;
    int32_t rows, cols;
    rc = tile_shape(pass, D, Hq, Hkv, &rows, &cols);
    if (rc) return rc;
    int64_t items = 0;
    for (int32_t s = 0; s < n; ++s) items += (cu[s + 1] - cu[s] + rows - 1) / rows;
    // a dK/dV list may hold split key tiles: every piece is one more item, every split tile one merge record
    const int32_t extra = pass == VA_PASS_BWD_DKDV ? max_partial_slots(D, Hkv) : 0;
    if ((items + extra) * works_per_item(pass, Hq, Hkv) > INT32_MAX / 2) return fail(VA_ESIZE, "va_worklist_size: too many works");
    *bytes = (size_t)worklist_layout(pass, D, Hq, Hkv, (int32_t)items + extra, extra / 2).total_recs * sizeof(WorkItem);
    return VA_OK;
}

int va_build_worklist(const int32_t* cu, const int32_t* prefix_lens, int32_t n,
                      int32_t mask_mode, int32_t pass, int32_t D, int32_t Hq, int32_t Hkv,
                      void* host_out, size_t bytes, int32_t* num_items) {
    if (!host_out || !num_items) return fail(VA_EINVAL, "va_build_worklist: null pointer");
    if (mask_mode < VA_MASK_CAUSAL || mask_mode > VA_MASK_SLIDING_WINDOW)
        return fail(VA_EUNSUPPORTED, "va_build_worklist: unknown mask mode %d", mask_mode);
    if (mask_mode != VA_MASK_CAUSAL && !prefix_lens)
        return fail(VA_EINVAL, "va_build_worklist: prefix mask needs prefix_lens");
    size_t need;
    int rc = va_worklist_size(cu, n, pass, D, Hq, Hkv, &need);
    if (rc) return rc;
    if (bytes < need) return fail(VA_ESIZE, "va_build_worklist: buffer of %zu bytes, need %zu", bytes, need);
    int32_t bm, bn;  // rows of an item, rows of the tiles it loops over
    tile_shape(pass, D, Hq, Hkv, &bm, &bn);

    std::vector<Keyed> items;
    std::vector<WorkItem> merges;
    // Forward and dQ: where every query tile of a sample costs the same (no causal structure: whole samples
    // visible), the plain order below already walks the tiles of a sample one after the other, i.e. is local by itself.
    bool tiles_differ = false;
    for (int32_t s = 0; s < n; ++s) {
        const int32_t c = cu[s], L = cu[s + 1] - c;
        int32_t P, P2;
        block_ends(prefix_lens, mask_mode, s, &P, &P2);
        if (!block_ends_valid(P, P2, L, mask_mode))
            return fail(VA_EINVAL, "va_build_worklist: block ends (%d, %d) of sample %d outside [0, %d] or out of order, or a window below 1",
                        P, P2, s, L);
        const int32_t Pm = P < 0 ? 0 : P, P2m = P2 < 0 ? 0 : P2;
        if (pass == VA_PASS_BWD_DKDV) {
            // item rows are key rows (bm), inner tiles are query tiles (bn)
            const int32_t q_tiles = (L + bn - 1) / bn;
            for (int32_t j0 = 0; j0 < L; j0 += bm) {
                int32_t first_row;  // first query row that sees key j0
                if (mask_mode == VA_MASK_CAUSAL || mask_mode == VA_MASK_SLIDING_WINDOW) first_row = j0;
                else if (j0 < Pm) first_row = 0;
                else if (mask_mode == VA_MASK_PREFIX_LM) first_row = Pm;
                else if (mask_mode == VA_MASK_THREE_BLOCK) first_row = j0 < P2m ? Pm : P2m;
                else first_row = j0;
                const int32_t qt_first = first_row / bn;
                int32_t qt_end = q_tiles;  // one past the last query tile with a row that sees a key of the tile
                if (mask_mode == VA_MASK_SLIDING_WINDOW) {
                    const int64_t last_row = std::min<int64_t>(L - 1, (int64_t)j0 + std::min(bm, L - j0) - 1 + Pm - 1);
                    qt_end = (int32_t)(last_row / bn) + 1;
                }
                WorkItem it = {{c + j0, std::min(bm, L - j0), c, qt_first, qt_end - qt_first, P2, P, L}};
                items.push_back({it.w[4], s, it});
            }
        } else {
            const size_t first_of_sample = items.size();
            for (int32_t r0 = 0; r0 < L; r0 += bm) {
                const int32_t rows = std::min(bm, L - r0);
                const int32_t kv_len = visible(r0 + rows - 1, L, Pm, P2m, mask_mode);
                const int32_t n_tiles = (kv_len + bn - 1) / bn;
                const int32_t n_full = visible(r0, L, Pm, P2m, mask_mode) / bn;
                WorkItem it = {{c + r0, rows, c, P2, n_full, n_tiles, P, L}};
                // under the sliding window the key tiles below the first row's window are not visited
                items.push_back({n_tiles - first_visible(r0, Pm, mask_mode) / bn, s, it});
                tiles_differ = tiles_differ || items.back().work != items[first_of_sample].work;
            }
        }
    }
    if (pass == VA_PASS_BWD_DKDV)
        split_late_tiles(items, merges, Hq / Hkv, Hkv, persistent_workgroups(pass, D), max_partial_slots(D, Hkv));
    sort_heaviest_first(items);
    const WorklistLayout lay = worklist_layout(pass, D, Hq, Hkv, (int32_t)items.size(), (int32_t)merges.size());
    WorkItem* out = static_cast<WorkItem*>(host_out);
    std::memset(out, 0, need);
    out[0] = {{kWorklistMagic, pass, bm, bn, D, mask_mode, lay.num_items, cu[n]}};
    out[1] = {{lay.num_workgroups, lay.num_works, lay.works_per_item, 0 /* flags, set below */, lay.table_rec, lay.id_rec,
               lay.total_recs, lay.num_merges}};
    for (size_t i = 0; i < items.size(); ++i) out[lay.item_rec + i] = items[i].it;
    for (size_t i = 0; i < merges.size(); ++i) out[lay.merge_rec + i] = merges[i];

    // Assignment of the works to the persistent workgroups.  cost(work) = its inner-loop steps plus a fixed
    // part; items are sorted by cost and every work of an item costs the same, so id order is cost order.
    const int32_t G = Hq / Hkv;
    const int32_t P = lay.num_workgroups;
    const int32_t per_item = lay.works_per_item;
    auto cost_of_item = [&](int32_t i) {
        return (int64_t)items[i].work * (pass == VA_PASS_BWD_DKDV ? G : 1) + kWorkFixedCost;
    };
    // the works in the order they are assigned, and the workgroup of each
    std::vector<int32_t> assigned, owner;
    assigned.reserve((size_t)lay.num_works);
    owner.reserve((size_t)lay.num_works);
    auto assign = [&](int32_t id, int32_t w) {
        assigned.push_back(id);
        owner.push_back(w);
    };
    struct Group {  // works of one (sample, KV head), or a part of them
        int64_t cost = 0;
        int32_t first = -1, last = -1;  // chain through next_in_group
    };
    std::vector<int32_t> next_in_group;
    auto append = [&](Group& g, int32_t id, int64_t cost) {
        g.cost += cost;
        if (g.first < 0) g.first = id;
        else next_in_group[g.last] = id;
        g.last = id;
    };
    // group indices, costliest first (ties: ascending), dealt to the XCDs, each to the least loaded one
    auto deal_to_xcds = [&](const std::vector<Group>& groups, std::vector<int32_t> (&of_xcd)[kXcds]) {
        std::vector<int32_t> order(groups.size());
        for (size_t i = 0; i < order.size(); ++i) order[i] = (int32_t)i;
        std::stable_sort(order.begin(), order.end(), [&](int32_t a, int32_t b) { return groups[a].cost > groups[b].cost; });
        int64_t xcd_load[kXcds] = {};
        for (int32_t gi : order) {
            int32_t x = 0;
            for (int32_t c = 1; c < kXcds; ++c)
                if (xcd_load[c] < xcd_load[x]) x = c;
            xcd_load[x] += groups[gi].cost;
            of_xcd[x].push_back(gi);
        }
    };
    if (tiles_differ && P % kXcds == 0) {
        // Forward and dQ: all works of one (sample, KV head) stream the same K and V rows.  Workgroup b runs
        // on XCD b % 8, and each XCD has an L2 of its own, so those works are given to workgroups of one XCD
        // and placed at about the same position of their queues: they then run at about the same time and
        // the rows are fetched into that L2 once instead of once per work.  Groups go to the XCDs, and
        // the works of a group to the workgroups of its XCD, longest processing time first; groups heavier
        // than a sixteenth of an XCD's share are cut into runs of consecutive query tiles first, so that
        // few heavy groups (one KV head, long samples) still balance.
        const int32_t chunks_per_head = per_item / Hkv;  // head chunks that share one KV head
        int64_t total = 0;
        for (int32_t i = 0; i < lay.num_items; ++i) total += cost_of_item(i) * per_item;
        const int64_t cap = std::max<int64_t>(1, total / (kXcds * 16));
        next_in_group.assign((size_t)lay.num_works, -1);
        std::vector<Group> groups;
        std::vector<int32_t> open((size_t)n * Hkv, -1);  // (sample, KV head) -> its current group
        for (int32_t i = 0; i < lay.num_items; ++i) {
            const int64_t cost = cost_of_item(i);
            for (int32_t chunk = 0; chunk < per_item; ++chunk) {
                int32_t& at = open[(size_t)items[i].sample * Hkv + chunk / chunks_per_head];
                if (at < 0 || groups[at].cost + cost > cap) {
                    at = (int32_t)groups.size();
                    groups.emplace_back();
                }
                append(groups[at], i * per_item + chunk, cost);
            }
        }
        std::vector<int32_t> of_xcd[kXcds];
        deal_to_xcds(groups, of_xcd);
        for (int32_t x = 0; x < kXcds; ++x) {
            LeastLoaded queue(x, P, kXcds);
            for (int32_t gi : of_xcd[x])
                for (int32_t id = groups[gi].first; id >= 0; id = next_in_group[id])
                    assign(id, queue.give(cost_of_item(id / per_item)));
        }
    } else if (pass == VA_PASS_BWD_DKDV) {
        // One work per workgroup; workgroup b of the launch runs on XCD b % 8 and takes the work at position b
        // of the id array.  Item order (heaviest first) balances best but spreads the key tiles of a sample
        // over all XCDs and over the run of the kernel, so that every tile fetches the sample's Q and dO rows
        // again (measured: 3.4 times the rows on heavy-tailed lengths).  The other order keeps the tiles of
        // one (sample, KV head) on one XCD, next to each other, heaviest sample first; the kernel walks the
        // query tiles downwards, so those tiles then read the same rows at the same time.  It is taken
        // where every workgroup slot runs at least four works (with one or two works per slot the tiles of a
        // sample run at the same time in either order, and item order measured 5 % faster) and a replay of the
        // hardware's dispatch says it ends within 3 % of the item order.
        std::vector<int32_t> order((size_t)lay.num_works);
        for (int32_t id = 0; id < lay.num_works; ++id) order[id] = id;
        if (P % kXcds == 0 && lay.num_works >= 4 * P) {
            next_in_group.assign((size_t)lay.num_works, -1);
            std::vector<Group> groups;
            std::vector<int32_t> index((size_t)n * Hkv, -1);  // (sample, KV head) -> group
            for (int32_t i = 0; i < lay.num_items; ++i) {
                const int64_t cost = cost_of_item(i);
                for (int32_t g = 0; g < per_item; ++g) {
                    int32_t& at = index[(size_t)items[i].sample * Hkv + g];
                    if (at < 0) {
                        at = (int32_t)groups.size();
                        groups.emplace_back();
                    }
                    append(groups[at], i * per_item + g, cost);
                }
            }
            std::vector<int32_t> of_xcd[kXcds], queue[kXcds];
            deal_to_xcds(groups, of_xcd);
            for (int32_t x = 0; x < kXcds; ++x)
                for (int32_t gi : of_xcd[x])
                    for (int32_t id = groups[gi].first; id >= 0; id = next_in_group[id]) queue[x].push_back(id);
            // position 8 k + x is the k-th work of XCD x; an XCD that has run out takes from the end of the
            // queue that has most left
            std::vector<int32_t> local;
            size_t head[kXcds] = {}, tail[kXcds];
            for (int32_t x = 0; x < kXcds; ++x) tail[x] = queue[x].size();
            for (int32_t pos = 0; pos < lay.num_works; ++pos) {
                const int32_t x = pos % kXcds;
                if (head[x] < tail[x]) {
                    local.push_back(queue[x][head[x]++]);
                    continue;
                }
                int32_t most = -1;
                for (int32_t c = 0; c < kXcds; ++c)
                    if (head[c] < tail[c] && (most < 0 || tail[c] - head[c] > tail[most] - head[most])) most = c;
                local.push_back(queue[most][--tail[most]]);
            }
            // replay of the dispatch: every XCD hands its positions, in order, to the least-loaded of its slots
            auto finish_time = [&](const std::vector<int32_t>& ord) {
                int64_t finish = 0;
                for (int32_t x = 0; x < kXcds; ++x) {
                    LeastLoaded slots(0, P / kXcds, 1);
                    for (int32_t pos = x; pos < lay.num_works; pos += kXcds) slots.give(cost_of_item(ord[pos] / per_item));
                    finish = std::max(finish, slots.last_finish());
                }
                return finish;
            };
            if (finish_time(local) * 100 <= finish_time(order) * 103) {
                order.swap(local);
                out[1].w[3] |= kListFlagInStep;
            }
        }
        // the table is not used by this pass; it holds the order in equal runs so that it still partitions the ids
        const int32_t per = std::max(1, (lay.num_works + P - 1) / P);
        for (int32_t i = 0; i < lay.num_works; ++i) assign(order[i], i / per);
    } else {
        // Longest processing time first: works in descending cost order (ties: ascending id), each to the
        // least-loaded workgroup (ties: lowest index).
        LeastLoaded queue(0, P, 1);
        for (int32_t id = 0; id < lay.num_works; ++id) assign(id, queue.give(cost_of_item(id / per_item)));
    }
    int32_t* table = out[lay.table_rec].w;
    int32_t* ids = out[lay.id_rec].w;
    std::vector<int32_t> at((size_t)P + 1, 0);  // first schedule position of each workgroup
    for (int32_t w : owner) ++at[(size_t)w + 1];
    for (int32_t w = 0; w < P; ++w) at[(size_t)w + 1] += at[w];
    for (int32_t w = 0; w < P; ++w) {
        int32_t* e = table + kTableWordsPerWorkgroup * w;
        e[10] = at[w];
        e[11] = at[(size_t)w + 1] - at[w];
    }
    for (size_t i = 0; i < assigned.size(); ++i) ids[at[owner[i]]++] = assigned[i];  // assignment order inside a workgroup
    for (int32_t w = 0; w < P; ++w) {
        int32_t* e = table + kTableWordsPerWorkgroup * w;
        if (e[11] == 0) continue;
        const int32_t* mine = ids + e[10];
        std::memcpy(e, items[mine[0] / per_item].it.w, 8 * sizeof(int32_t));
        e[8] = mine[0];
        e[9] = mine[e[11] > 1 ? 1 : 0];
    }
    *num_items = lay.num_items;
    return VA_OK;
}

// bfloat16 bits -> float
static inline float bf16_to_float(uint16_t b) {
    uint32_t u = (uint32_t)b << 16;
    float f;
    std::memcpy(&f, &u, 4);
    return f;
}

// Round-to-nearest-even E4M3 (OCP, "fn": no infinities, NaN = 0x7F), saturating.
static inline uint8_t encode_e4m3(float x) {
    if (std::isnan(x)) return 0x7F;
    const uint8_t sign = std::signbit(x) ? 0x80 : 0x00;
    const float a = std::fabs(x);
    if (a >= 448.0f) return sign | 0x7E;
    if (a < 0.015625f) {  // below 2^-6: subnormal spacing 2^-9; a result of 8 is the first normal
        return sign | (uint8_t)std::nearbyintf(a * 512.0f);
    }
    int e;
    const float frac = std::frexp(a, &e);  // a = frac * 2^e, frac in [0.5, 1)
    int m = (int)std::nearbyintf((frac * 2.0f - 1.0f) * 8.0f);
    e -= 1;
    if (m == 8) {
        m = 0;
        e += 1;
    }
    return sign | (uint8_t)(((e + 7) << 3) | m);
}

int va_quantize_e4m3_per_head(const uint16_t* x, int32_t T, int32_t H, int32_t D,
                              uint8_t* codes, float* descale) {
    if (T < 0 || H <= 0 || D <= 0 || !descale || (T > 0 && (!x || !codes)))
        return fail(VA_EINVAL, "va_quantize_e4m3_per_head: null pointer or bad size");
    std::vector<float> amax((size_t)H, 0.0f);
    for (int64_t t = 0; t < T; ++t)
        for (int32_t h = 0; h < H; ++h) {
            const uint16_t* row = x + ((size_t)t * H + h) * D;
            float m = amax[h];
            for (int32_t d = 0; d < D; ++d) m = std::max(m, std::fabs(bf16_to_float(row[d])));
            amax[h] = m;
        }
    for (int32_t h = 0; h < H; ++h) {
        const float s = amax[h] / 448.0f;
        descale[h] = s > 0.0f ? s : 1.0f;
    }
    for (int64_t t = 0; t < T; ++t)
        for (int32_t h = 0; h < H; ++h) {
            const size_t base = ((size_t)t * H + h) * D;
            for (int32_t d = 0; d < D; ++d) codes[base + d] = encode_e4m3(bf16_to_float(x[base + d]) / descale[h]);
        }
    return VA_OK;
}

int va_quantize_e4m3_blockwise(const uint16_t* x, const int32_t* cu_seqlens, int32_t num_seqs, int32_t H, int32_t D,
                               uint8_t* codes, float* descale_tok) {
    const char* who = "va_quantize_e4m3_blockwise";
    if (!cu_seqlens || num_seqs < 0 || H <= 0 || D <= 0) return fail(VA_EINVAL, "%s: null pointer or bad size", who);
    if (cu_seqlens[0] != 0) return fail(VA_EINVAL, "%s: cu_seqlens[0] must be 0", who);
    for (int32_t s = 0; s < num_seqs; ++s)
        if (cu_seqlens[s + 1] < cu_seqlens[s]) return fail(VA_EINVAL, "%s: cu_seqlens decreases at %d", who, s);
    const int32_t T = cu_seqlens[num_seqs];
    if (T > 0 && (!x || !codes || !descale_tok)) return fail(VA_EINVAL, "%s: null buffer", who);
    for (int32_t s = 0; s < num_seqs; ++s)
        for (int32_t r0 = cu_seqlens[s]; r0 < cu_seqlens[s + 1]; r0 += VA_FP8_BLOCK_TOKENS) {
            const int32_t r1 = std::min(cu_seqlens[s + 1], r0 + VA_FP8_BLOCK_TOKENS);
            for (int32_t h = 0; h < H; ++h) {
                float amax = 0.0f;
                for (int32_t t = r0; t < r1; ++t) {
                    const uint16_t* row = x + ((size_t)t * H + h) * D;
                    for (int32_t d = 0; d < D; ++d) amax = std::max(amax, std::fabs(bf16_to_float(row[d])));
                }
                const float sc = amax / 448.0f;
                const float descale = sc > 0.0f ? sc : 1.0f;
                for (int32_t t = r0; t < r1; ++t) {
                    const size_t base = ((size_t)t * H + h) * D;
                    descale_tok[(size_t)t * H + h] = descale;
                    for (int32_t d = 0; d < D; ++d) codes[base + d] = encode_e4m3(bf16_to_float(x[base + d]) / descale);
                }
            }
        }
    return VA_OK;
}

}  // extern "C"
