// Host side of the batched counts: planning of the items, launch groups (one
// per distinct binning), the workgroups' shares by estimated cost, sorted-order
// mask bits, the device counts, and the HIP graph that replays the launches.
#include <string.h>

#include <algorithm>
#include <cmath>
#include <numeric>
#include <vector>

#include "cute_internal.h"
#include "runtime.h"

using namespace cute;

namespace {

// Items of one binning, counted by one persistent launch.
struct Group {
    Plan pl;
    int prec = 0;                    // precision path of the launch (plan_form)
    int grid = 0;                    // workgroups
    BatchArgs ba;                    // device pointers filled at creation
    std::vector<int> items;          // item indices, largest estimated cost first
};

}  // namespace

struct cute_batch {
    int device = -1;                 // where its memory lies (-1: none yet)
    int prec = 0;
    int n_items = 0;
    std::vector<Group> groups;
    std::vector<int64_t> words;      // count words per item
    std::vector<int64_t> offset;     // offset of each item's counts
    int64_t total_words = 0;
    unsigned long long* work = nullptr;   // counts | stats (4 per item) | heads (1 per item) | done (1 per group)
    size_t work_words = 0;
    CountArgs* dargs = nullptr;      // one per item
    uint32_t* dntiles = nullptr;     // per item: home tiles, log2 of their parts
    std::vector<void*> owned;        // device allocations (stream-ordered)
    hipStream_t cap = nullptr;       // private stream used for capture
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
};

namespace {

template <typename T>
cute_status owned_alloc(cute_batch* b, T** p, size_t count, hipStream_t s) {
    cute_status st = dalloc(p, count, s);
    if (st == CUTE_OK) b->owned.push_back(*p);
    return st;
}

void release(cute_batch* b) {
    if (!b) return;
    // the batch's device, whatever device is current: its work ends, and its
    // memory goes back to that device's pool
    int cur = -1;
    const bool other = b->device >= 0 && hipGetDevice(&cur) == hipSuccess && cur != b->device;
    if (other) (void)hipSetDevice(b->device);
    (void)hipDeviceSynchronize();
    if (b->exec) (void)hipGraphExecDestroy(b->exec);
    if (b->graph) (void)hipGraphDestroy(b->graph);
    if (b->cap) (void)hipStreamDestroy(b->cap);
    for (void* p : b->owned) dfree(p, nullptr);
    if (other) (void)hipSetDevice(cur);
    delete b;
}

// Enqueue one run: clear counts, statistics and task heads, then one
// persistent launch per group. No allocation, memset or synchronisation.
cute_status enqueue_run(cute_batch* b, hipStream_t s) {
    cute_status st = zero_u64(b->work, b->work_words, s);
    if (st != CUTE_OK) return st;
    for (const Group& g : b->groups) {
        if (g.ba.nlist == 0) continue;
        st = batch_launch(g.ba, g.pl.mode, g.prec, g.pl.est, g.grid, g.pl.lds, s);
        if (st != CUTE_OK) return st;
    }
    return CUTE_OK;
}

// graph: capture a run for CUTE_BATCH_GRAPH (a batch that runs once is not
// worth its capture).
cute_status create(const cute_batch_item* items, int32_t n_items, cute_precision prec,
                   hipStream_t hs, bool graph, cute_batch* b) {
    cute_status s;
    if (prec != CUTE_PREC_FP64 && prec != CUTE_PREC_FP32_EDGE && prec != CUTE_PREC_FP32_ONLY)
        return fail(CUTE_E_INVALID_ARG, "unknown precision");
    b->prec = (int)prec;
    b->n_items = n_items;
    std::vector<ItemGeom> geo(n_items);
    std::vector<int> gid(n_items, -1);
    // ---- validate and group the items by binning ---------------------------
    for (int i = 0; i < n_items; i++) {
        const cute_batch_item& it = items[i];
        if (!it.a) return fail(CUTE_E_INVALID_ARG, "item " + std::to_string(i) + ": grid a is NULL");
        if ((s = validate_binning(it.bins)) != CUTE_OK) return s;
        const bool is_auto = it.b == nullptr || it.b == it.a;
        const cute_grid* gb = is_auto ? it.a : it.b;
        if (it.a->h.wt != nullptr || gb->h.wt != nullptr)
            return fail(CUTE_E_UNSUPPORTED, "item " + std::to_string(i) + ": pixel maps are counted one at a time");
        int g = -1;
        for (size_t k = 0; k < b->groups.size(); k++) {
            const int first = b->groups[k].items[0];
            if (same_binning(items[first].bins, it.bins)) {
                g = (int)k;
                break;
            }
        }
        if (g < 0) {
            b->groups.emplace_back();
            g = (int)b->groups.size() - 1;
            plan_binning(it.bins, b->groups[g].pl);
        }
        Group& G = b->groups[g];
        if ((s = plan_item(it.a->h, gb->h, is_auto, it.bins, G.pl, &geo[i])) != CUTE_OK) {
            set_error("item " + std::to_string(i) + ": " + std::string(cute_last_error()));
            return s;
        }
        G.items.push_back(i);
        gid[i] = g;
        const int64_t w = (int64_t)G.pl.a.nbins;
        b->words.push_back(w);
        b->offset.push_back(b->total_words);
        b->total_words += w;
    }
    // ---- bands (one error model per group), LDS plan, kernel attributes -----
    int dev = 0, ncu = 0;
    if ((s = ensure_device_ready(&dev)) != CUTE_OK) return s;
    // the set-up work on hs (and every replay, which follows it) comes after
    // the builds of the grids
    for (int i = 0; i < n_items; i++) {
        if ((s = grid_wait(items[i].a, hs)) != CUTE_OK) return s;
        if (items[i].b && items[i].b != items[i].a && (s = grid_wait(items[i].b, hs)) != CUTE_OK)
            return s;
    }
    b->device = dev;
    CUTE_HIP(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
    for (Group& G : b->groups) {
        FormErr em = geo[G.items[0]].em;
        for (int i : G.items) em = max_err(em, geo[i].em);
        G.prec = plan_form(items[G.items[0]].bins, em, b->prec, G.pl);
        if ((s = plan_lds(G.pl, 16, &G.prec)) != CUTE_OK) return s;
        int per_cu = 1;
        if ((s = batch_prepare(G.pl.mode, G.prec, G.pl.est, G.pl.lds, &per_cu)) != CUTE_OK) return s;
        G.grid = per_cu * ncu;
        std::stable_sort(G.items.begin(), G.items.end(),
                         [&](int x, int y) { return geo[x].cost > geo[y].cost; });
    }
    // ---- per item: slots of its tiles, mask bits -------------------------------
    // Tiles are built into slots without a wait for their count, as a single
    // count does; only for very sparse grids they are counted first.
    struct ItemTiles {
        Tile *built = nullptr, *out = nullptr;   // counted tiles (sparse grids), the ordered list
        uint32_t n = 0;                          // slots
        double est = 0.0;                        // estimated tiles
        PartCost pc{1u, 0.f, 0.f, 0.f};          // the item's share of its launch's waves
    };
    std::vector<ItemTiles> it_tiles(n_items);
    std::vector<CountArgs> args(n_items);
    TempList tmp(hs);
    size_t max_slots = 1;
    for (int i = 0; i < n_items; i++) {
        const cute_batch_item& it = items[i];
        const bool is_auto = it.b == nullptr || it.b == it.a;
        const GridHost& A = it.a->h;
        const GridHost& B = is_auto ? it.a->h : it.b->h;
        ItemTiles& t = it_tiles[i];
        if (A.n > 0 && B.n > 0) {
            const uint64_t min_tiles = ((uint64_t)A.n + A.tile_max - 1) / A.tile_max;
            const uint64_t bound = tile_count_bound(A, geo[i].max_w);
            // (the ordered list keeps a slot per possible tile for the batch's
            // life: at most eight times what the points need and 32 KB, where a
            // single count accepts 1 MB for its own duration)
            if (bound <= 8 * min_tiles + 2048 && bound < (uint64_t(1) << 31)) {
                t.n = (uint32_t)bound;
                t.est = std::sqrt((double)min_tiles * (double)bound);
                max_slots = std::max<size_t>(max_slots, t.n);
            } else {
                if ((s = build_tiles(A, geo[i].max_w, hs, &t.built, &t.n)) != CUTE_OK) return s;
                tmp.ptrs.push_back(t.built);
                t.est = (double)t.n;
                max_slots = std::max<size_t>(max_slots, t.n);
            }
            if ((s = owned_alloc(b, &t.out, (size_t)t.n, hs)) != CUTE_OK) return s;
        }
        CountArgs& a = args[i];
        a = b->groups[gid[i]].pl.a;
        apply_item(geo[i], &a);
        // masks -> sorted-order bits
        const uint8_t* masks[2] = {it.mask_a, is_auto ? nullptr : it.mask_b};
        const GridHost* gh[2] = {&A, &B};
        const uint32_t* bits[2] = {nullptr, nullptr};
        for (int side = 0; side < 2; side++) {
            if (!masks[side] || gh[side]->n == 0) continue;
            const size_t n = (size_t)gh[side]->n;
            uint32_t* mb = nullptr;
            if ((s = owned_alloc(b, &mb, (n + 31) / 32, hs)) != CUTE_OK) return s;
            const uint8_t* src = masks[side];
            uint8_t* dm = nullptr;
            if (!it.masks_on_device) {
                if ((s = dalloc(&dm, n, hs)) != CUTE_OK) return s;
                const hipError_t e = hipMemcpyAsync(dm, src, n, hipMemcpyHostToDevice, hs);
                if (e != hipSuccess) {
                    dfree(dm, hs);
                    return hip_status(e, "mask copy");
                }
                src = dm;
            }
            s = mask_bits(src, *gh[side], mb, hs);
            if (dm) dfree(dm, hs);
            if (s != CUTE_OK) return s;
            bits[side] = mb;
        }
        a.mbA = bits[0];
        a.mbB = is_auto ? bits[0] : bits[1];
    }
    // ---- one device block, filled by one copy ----------------------------------
    // [per group: T1 | T2 | B1 | B2 | items, largest first | first item of each
    //  workgroup] [per item: stencil] [arguments] [tiles and parts per item, overflow flag,
    //  bucket counts of the tile orders: zero]
    std::vector<unsigned char> img;
    auto put = [&](const void* p, size_t bytes) {
        const size_t o = img.size();
        img.resize(o + ((bytes + 15) & ~(size_t)15));
        if (bytes) memcpy(img.data() + o, p, bytes);
        return o;
    };
    struct GroupOff {
        size_t t1, t2, b1, b2, list, first;
    };
    std::vector<GroupOff> go(b->groups.size());
    for (size_t gi = 0; gi < b->groups.size(); gi++) {
        Group& G = b->groups[gi];
        std::vector<uint32_t> list, first;
        std::vector<double> cost;
        double tiles = 0.0, slots = 0.0, homes = 0.0, near = 0.0;
        for (int i : G.items) {
            if (it_tiles[i].n == 0) continue;
            list.push_back((uint32_t)i);
            cost.push_back(std::max(geo[i].cost, 1.0));
            tiles += it_tiles[i].est;
            slots += (double)it_tiles[i].n;
            homes += (double)items[i].a->h.n;
            near += geo[i].near * (double)items[i].a->h.n;
        }
        // (an estimate of the parts for the size of the launch; the cut itself is
        // made on the device, by the tiles' costs)
        const int plog = homes > 0.0 ? part_log(2.0 * tiles, near / homes, ncu) : 0;
        const double tasks = slots * (double)(1 << plog);
        G.grid = (int)std::max(1.0, std::min((double)G.grid, std::ceil(tasks / kWgWaves)));
        if (!list.empty()) first = batch_first(cost, G.grid);
        double all = 0.0;
        for (double c : cost) all += c;
        for (size_t k = 0; k < list.size(); k++)
            it_tiles[list[k]].pc =
                part_cost(G.pl, G.prec, (uint32_t)std::ceil((double)(G.grid * kWgWaves) * cost[k] / all));
        go[gi].t1 = put(G.pl.T1.data(), G.pl.T1.size() * 8);
        go[gi].t2 = put(G.pl.T2.data(), G.pl.T2.size() * 8);
        go[gi].b1 = put(G.pl.band1.data(), G.pl.band1.size() * 8);
        go[gi].b2 = put(G.pl.band2.data(), G.pl.band2.size() * 8);
        go[gi].list = put(list.data(), list.size() * 4);
        go[gi].first = put(first.data(), first.size() * 4);
        memset(&G.ba, 0, sizeof(G.ba));
        G.ba.nlist = (uint32_t)list.size();
    }
    std::vector<size_t> so(n_items);
    for (int i = 0; i < n_items; i++) so[i] = put(geo[i].stencil.data(), geo[i].stencil.size() * sizeof(int4));
    const size_t oAR = img.size();
    const size_t oNT = oAR + ((sizeof(CountArgs) * (size_t)n_items + 15) & ~(size_t)15);
    const size_t oHI = oNT + ((2 * (size_t)n_items + 1) * 4 + 15) / 16 * 16;
    const size_t total = oHI + (size_t)n_items * kTileBuckets * 4;
    img.resize(total, 0);
    unsigned char* blob = nullptr;
    b->work_words = (size_t)b->total_words + 5 * (size_t)n_items + b->groups.size();
    if ((s = owned_alloc(b, &blob, total, hs)) != CUTE_OK) return s;
    if ((s = owned_alloc(b, &b->work, b->work_words, hs)) != CUTE_OK) return s;
    b->dargs = reinterpret_cast<CountArgs*>(blob + oAR);
    b->dntiles = reinterpret_cast<uint32_t*>(blob + oNT);
    for (int i = 0; i < n_items; i++) {
        const GroupOff& g = go[gid[i]];
        CountArgs& a = args[i];
        a.T1 = reinterpret_cast<const double*>(blob + g.t1);
        a.T2 = reinterpret_cast<const double*>(blob + g.t2);
        a.band1 = reinterpret_cast<const float2*>(blob + g.b1);
        a.band2 = reinterpret_cast<const float2*>(blob + g.b2);
        a.self = b->dargs + i;
        a.counts = b->work + b->offset[i];
        a.stats = b->work + b->total_words + 4 * (size_t)i;
        a.nst = (int)geo[i].stencil.size();
        a.stencil = a.nst > 0 ? reinterpret_cast<const int4*>(blob + so[i]) : nullptr;
        a.tiles = it_tiles[i].out;
        a.ntiles = it_tiles[i].n;
        memcpy(img.data() + oAR + sizeof(CountArgs) * (size_t)i, &a, sizeof(a));
    }
    for (size_t gi = 0; gi < b->groups.size(); gi++) {
        Group& G = b->groups[gi];
        BatchArgs& ba = G.ba;
        ba.items = b->dargs;
        ba.list = reinterpret_cast<const uint32_t*>(blob + go[gi].list);
        ba.first = reinterpret_cast<const uint32_t*>(blob + go[gi].first);
        ba.ntiles = b->dntiles;
        ba.heads = b->work + b->total_words + 4 * (size_t)n_items;
        ba.done = ba.heads + n_items + gi;
        ba.n1 = G.pl.a.n1;
        ba.n2 = G.pl.a.n2;
        ba.nbins = G.pl.a.nbins;
        ba.copies = G.pl.a.copies;
        ba.hist_words = G.pl.a.hist_words;
        ba.T1 = reinterpret_cast<const double*>(blob + go[gi].t1);
        ba.T2 = reinterpret_cast<const double*>(blob + go[gi].t2);
        ba.band1 = reinterpret_cast<const float2*>(blob + go[gi].b1);
        ba.band2 = reinterpret_cast<const float2*>(blob + go[gi].b2);
    }
    CUTE_HIP(hipMemcpyAsync(blob, img.data(), total, hipMemcpyHostToDevice, hs));
    // ---- the tiles, heavy ones first within each item ---------------------------
    // (one set of slots, keys and ranks for all items: the stream orders them)
    Tile* slots = nullptr;
    uint32_t* keys = nullptr;
    if ((s = tmp.alloc(&slots, max_slots)) != CUTE_OK) return s;
    if ((s = tmp.alloc(&keys, 2 * max_slots)) != CUTE_OK) return s;
    uint32_t* overflow = b->dntiles + 2 * (size_t)n_items;
    for (int i = 0; i < n_items; i++) {
        const ItemTiles& t = it_tiles[i];
        if (t.n == 0) continue;
        if (!t.built && (s = tiles_to_slots(items[i].a->h, geo[i].max_w, t.n, slots, overflow, nullptr, hs)) != CUTE_OK)
            return s;
        if ((s = order_tiles_to(args[i], t.built ? t.built : slots, t.n, t.pc, keys, keys + max_slots,
                                reinterpret_cast<uint32_t*>(blob + oHI) + (size_t)i * kTileBuckets, t.out,
                                b->dntiles + 2 * (size_t)i, hs)) != CUTE_OK)
            return s;
    }
    uint32_t over = 0;
    CUTE_HIP(hipMemcpyAsync(&over, overflow, sizeof(over), hipMemcpyDeviceToHost, hs));
    CUTE_HIP(hipStreamSynchronize(hs));
    if (over) return fail(CUTE_E_INTERNAL, "tile slots overflowed");
    if (!graph) return CUTE_OK;
    // ---- capture one run in a graph ----------------------------------------------
    CUTE_HIP(hipStreamCreateWithFlags(&b->cap, hipStreamNonBlocking));
    CUTE_HIP(hipStreamBeginCapture(b->cap, hipStreamCaptureModeThreadLocal));
    s = enqueue_run(b, b->cap);
    hipGraph_t g = nullptr;
    hipError_t e = hipStreamEndCapture(b->cap, &g);
    if (s != CUTE_OK) {
        if (g) (void)hipGraphDestroy(g);
        return s;
    }
    if (e != hipSuccess) return hip_status(e, "hipStreamEndCapture");
    b->graph = g;
    CUTE_HIP(hipGraphInstantiate(&b->exec, b->graph, nullptr, nullptr, 0));
    return CUTE_OK;
}

}  // namespace

static cute_status batch_create(const cute_batch_item* items, int32_t n_items, cute_precision prec,
                                void* stream, bool graph, cute_batch** out) {
    *out = nullptr;
    if (!items || n_items < 1) return fail(CUTE_E_INVALID_ARG, "no items");
    cute_batch* b = new cute_batch();
    cute_status s = create(items, n_items, prec, (hipStream_t)stream, graph, b);
    if (s != CUTE_OK) {
        (void)hipStreamSynchronize((hipStream_t)stream);
        release(b);
        return s;
    }
    *out = b;
    return CUTE_OK;
}

extern "C" cute_status cute_batch_create(const cute_batch_item* items, int32_t n_items,
                                         cute_precision prec, void* stream, cute_batch** out) {
    if (!out) return fail(CUTE_E_INVALID_ARG, "out is NULL");
    return batch_create(items, n_items, prec, stream, true, out);
}

extern "C" cute_status cute_batch_run(cute_batch* b, int32_t flags, void* stream) {
    if (!b) return fail(CUTE_E_INVALID_ARG, "batch is NULL");
    hipStream_t hs = (hipStream_t)stream;
    if (flags == CUTE_BATCH_EAGER) return enqueue_run(b, hs);
    if (flags != CUTE_BATCH_GRAPH) return fail(CUTE_E_INVALID_ARG, "unknown flags");
    CUTE_HIP(hipGraphLaunch(b->exec, hs));
    return CUTE_OK;
}

extern "C" cute_status cute_batch_layout(const cute_batch* b, int32_t item, int64_t* words,
                                         int64_t* offset) {
    if (!b) return fail(CUTE_E_INVALID_ARG, "batch is NULL");
    if (item < -1 || item >= b->n_items) return fail(CUTE_E_INVALID_ARG, "item out of range");
    if (words) *words = item < 0 ? b->total_words : b->words[item];
    if (offset) *offset = item < 0 ? 0 : b->offset[item];
    return CUTE_OK;
}

extern "C" cute_status cute_batch_counts(const cute_batch* b, int32_t item, uint64_t* out,
                                         int32_t on_device, void* stream) {
    if (!b || !out) return fail(CUTE_E_INVALID_ARG, "NULL argument");
    if (item < -1 || item >= b->n_items) return fail(CUTE_E_INVALID_ARG, "item out of range");
    hipStream_t hs = (hipStream_t)stream;
    const int64_t w = item < 0 ? b->total_words : b->words[item];
    const int64_t o = item < 0 ? 0 : b->offset[item];
    CUTE_HIP(hipMemcpyAsync(out, b->work + o, (size_t)w * 8,
                            on_device ? hipMemcpyDeviceToDevice : hipMemcpyDeviceToHost, hs));
    if (!on_device) CUTE_HIP(hipStreamSynchronize(hs));
    return CUTE_OK;
}

// Statistics of an item (or all) from the work area and the tile counts on the
// host.
static cute_status batch_stats(const cute_batch* b, int32_t item, const unsigned long long* h,
                               const uint32_t* ntiles, cute_count_stats* st) {
    memset(st, 0, sizeof(*st));
    bool complete = true;
    for (int i = 0; i < b->n_items; i++) {
        if (item >= 0 && i != item) continue;
        const unsigned long long* sv = h + b->total_words + 4 * (size_t)i;
        st->pair_evals += sv[0];
        st->retests += sv[1];
        st->flips += sv[2];
        st->tiles += sv[3];
        for (int64_t k = 0; k < b->words[i]; k++) st->pairs_in_range += h[b->offset[i] + k];
        complete = complete && sv[3] == ntiles[2 * (size_t)i];
    }
    if (!complete) return fail(CUTE_E_INTERNAL, "not every tile was processed");
    return CUTE_OK;
}

extern "C" cute_status cute_batch_stats(const cute_batch* b, int32_t item, cute_count_stats* st,
                                        void* stream) {
    if (!b || !st) return fail(CUTE_E_INVALID_ARG, "NULL argument");
    if (item < -1 || item >= b->n_items) return fail(CUTE_E_INVALID_ARG, "item out of range");
    hipStream_t hs = (hipStream_t)stream;
    std::vector<unsigned long long> h(b->work_words);
    std::vector<uint32_t> nt(2 * (size_t)b->n_items);
    CUTE_HIP(hipMemcpyAsync(h.data(), b->work, b->work_words * 8, hipMemcpyDeviceToHost, hs));
    CUTE_HIP(hipMemcpyAsync(nt.data(), b->dntiles, nt.size() * 4, hipMemcpyDeviceToHost, hs));
    CUTE_HIP(hipStreamSynchronize(hs));
    return batch_stats(b, item, h.data(), nt.data(), st);
}

extern "C" void cute_batch_free(cute_batch* b) { release(b); }

extern "C" cute_status cute_count_pairs_batched(const cute_batch_item* items, int32_t n_items,
                                                cute_precision prec, uint64_t* const* counts,
                                                int32_t counts_on_device, cute_count_stats* st,
                                                void* stream) {
    if (!counts) return fail(CUTE_E_INVALID_ARG, "counts is NULL");
    for (int i = 0; i < n_items; i++)
        if (!counts[i]) return fail(CUTE_E_INVALID_ARG, "counts[" + std::to_string(i) + "] is NULL");
    cute_batch* b = nullptr;
    cute_status s = batch_create(items, n_items, prec, stream, false, &b);
    if (s != CUTE_OK) return s;
    hipStream_t hs = (hipStream_t)stream;
    auto run = [&]() -> cute_status {
        cute_status r;
        EventTimer timer(hs);
        if ((r = enqueue_run(b, hs)) != CUTE_OK) return r;
        timer.stop();
        if (counts_on_device)
            for (int i = 0; i < n_items; i++)
                if ((r = cute_batch_counts(b, i, counts[i], 1, stream)) != CUTE_OK) return r;
        // counts, statistics and tile counts in one wait, through pinned memory
        // unless they are large
        const size_t wb = b->work_words * 8, bytes = wb + (size_t)n_items * 8;
        HostStage stage(hs);
        std::vector<unsigned char> pageable;
        unsigned char* hb = nullptr;
        if (bytes > ((size_t)8 << 20)) {
            pageable.resize(bytes);
            hb = pageable.data();
        } else if ((r = stage.get(bytes, &hb)) != CUTE_OK) {
            return r;
        }
        CUTE_HIP(hipMemcpyAsync(hb, b->work, wb, hipMemcpyDeviceToHost, hs));
        CUTE_HIP(hipMemcpyAsync(hb + wb, b->dntiles, (size_t)n_items * 8, hipMemcpyDeviceToHost, hs));
        CUTE_HIP(hipStreamSynchronize(hs));
        const unsigned long long* h = reinterpret_cast<const unsigned long long*>(hb);
        if (!counts_on_device)
            for (int i = 0; i < n_items; i++) memcpy(counts[i], h + b->offset[i], (size_t)b->words[i] * 8);
        cute_count_stats all;
        r = batch_stats(b, -1, h, reinterpret_cast<const uint32_t*>(hb + wb), &all);
        all.ms_count = timer.elapsed_ms();
        if (st) *st = all;
        return r;
    };
    s = run();
    cute_batch_free(b);
    return s;
}
