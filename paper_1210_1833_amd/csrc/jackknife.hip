// Jackknife pair counts by region decomposition.
//
// With K regions, the jackknife catalog k is the whole catalog without the
// points of region k. Its autocorrelation is the total minus T_k, the pairs
// with at least one point in region k (counted once). One pass gives every
// T_k and the total: over the full stencil (every ordered pair (i, j), i != j,
// visited once from its first point) region a's histogram collects S_a = 2 H_aa,
// the pairs with both points in it, in the low halves of its 64-bit counters
// and D_a = sum_{b != a} H_ab in the high ones (H_ab: unordered pairs between
// regions a and b; a same-region pair is visited from both of its points).
// T_a = S_a / 2 + D_a, and the total is half the sum of all S_a + D_a. The cost
// is about two counts of the catalog, whatever K, instead of K masked counts.
// (The midpoint kinds have 32-bit counters: a pair adds 1 or 2 to them, which
// makes 2 T_a, and the total is one more autocorrelation; so is FP32_ONLY's,
// whose decision of a pair may depend on the point it is counted from.)
//
// A cross-correlation (catalogs A and B, each with its regions) works the
// same way with two passes: pairs whose A point lies in region k (A homes,
// weight 1) plus pairs whose B point lies in region k and whose A point does
// not (B homes, A neighbours, weight 0 for a neighbour in the home region and
// 1 otherwise) make T_k, and jack_k = total - T_k; the first pass visits every
// pair once, so its sum is the total (except FP32_ONLY, as above). Pair
// separations are symmetric, so a pair counted from its B point lands in the
// same bin.
//
// A pass runs on a copy of the home grid whose points are sorted by region
// inside each cell (the cells and their offsets are unchanged), so that home
// tiles hold a single region; the tiles of one region form one item of a
// batched launch, whose workgroup histogram then always belongs to one
// region.
#include <hipcub/hipcub.hpp>
#include <string.h>

#include <algorithm>
#include <vector>

#include "cute_internal.h"
#include "runtime.h"

using namespace cute;

namespace {

// key (cell, region) of every sorted point; one thread per point, which looks
// its cell up among the cells' offsets (a thread per cell walked its points one
// after the other: 81 us for 2.5e5 points, 7 so)
template <typename Key>
__global__ __launch_bounds__(256) void k_region_keys(const uint32_t* __restrict__ cs, uint32_t ncells,
                                                     uint32_t n, const P64* __restrict__ p64,
                                                     const int32_t* __restrict__ region,
                                                     uint32_t K, Key* __restrict__ key,
                                                     uint32_t* __restrict__ perm,
                                                     uint32_t* __restrict__ bad) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int32_t r = region[p64[i].idx];
    const bool ok = r >= 0 && (uint32_t)r < K;
    if (!ok) atomicOr(bad, 1u);
    uint32_t lo = 0, hi = ncells;   // cs[lo] <= i < cs[hi]
    while (hi - lo > 1u) {
        const uint32_t m = (lo + hi) >> 1;
        if (cs[m] <= i) lo = m; else hi = m;
    }
    key[i] = (Key)lo * (Key)K + (Key)(ok ? (uint32_t)r : 0u);
    perm[i] = i;
}

// the grid copy in (cell, region) order, each point's region, and its region
// and cell along x in one word
template <typename Key>
__global__ __launch_bounds__(256) void k_region_gather(uint32_t n, const uint32_t* __restrict__ perm,
                                                       const Key* __restrict__ key, uint32_t K, uint32_t nx,
                                                       const float4* __restrict__ p32,
                                                       const P64* __restrict__ p64,
                                                       float4* __restrict__ q32, P64* __restrict__ q64,
                                                       uint32_t* __restrict__ rc,
                                                       uint16_t* __restrict__ reg) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint32_t j = perm[i];
    q32[i] = p32[j];
    q64[i] = p64[j];
    const Key k = key[i];
    const uint32_t r = (uint32_t)(k % K), c = (uint32_t)(k / K) % nx;
    reg[i] = (uint16_t)r;
    rc[i] = (r << 16) | c;
}

}  // namespace

namespace {

// A grid copy whose points are in (cell, region) order, in stream-ordered
// temporary memory, with the region of each point.
struct RegionCopy {
    GridHost R;
    uint16_t* regs = nullptr;
    uint32_t* rc = nullptr;    // region << 16 | cell along x
    uint32_t* bad = nullptr;   // nonzero when a label was out of range (read in region_pass)
};

template <typename Key>
cute_status region_sort(const GridHost& G, const int32_t* dreg, uint32_t ncells, int32_t K, hipStream_t hs,
                        TempList& tmp, RegionCopy* out) {
    cute_status s;
    const size_t n = (size_t)G.n;
    const unsigned nb = (unsigned)((n + 255) / 256);
    Key* k = nullptr;
    uint32_t* v = nullptr;
    if ((s = tmp.alloc(&k, 2 * n)) != CUTE_OK) return s;
    if ((s = tmp.alloc(&v, 2 * n)) != CUTE_OK) return s;
    hipLaunchKernelGGL(k_region_keys<Key>, dim3(nb), dim3(256), 0, hs, G.cstart, ncells, (uint32_t)n, G.p64,
                       dreg, (uint32_t)K, k, v, out->bad);
    CUTE_HIP(hipGetLastError());
    int bits = 1;
    while (bits < 64 && (((uint64_t)ncells * (uint64_t)K) >> bits) != 0) bits++;
    size_t tb = 0;
    CUTE_HIP(hipcub::DeviceRadixSort::SortPairs(nullptr, tb, k, k + n, v, v + n, (int)n, 0, bits, hs));
    unsigned char* tsort = nullptr;
    if ((s = tmp.alloc(&tsort, tb)) != CUTE_OK) return s;
    CUTE_HIP(hipcub::DeviceRadixSort::SortPairs(tsort, tb, k, k + n, v, v + n, (int)n, 0, bits, hs));
    hipLaunchKernelGGL(k_region_gather<Key>, dim3(nb), dim3(256), 0, hs, (uint32_t)n, v + n, k + n, (uint32_t)K,
                       (uint32_t)G.nx, G.p32, G.p64, out->R.p32, out->R.p64, out->rc, out->regs);
    CUTE_HIP(hipGetLastError());
    return CUTE_OK;
}

cute_status region_copy(const GridHost& G, const int32_t* region, int32_t regions_on_device,
                        int32_t K, hipStream_t hs, TempList& tmp, RegionCopy* out) {
    cute_status s;
    const int64_t n = G.n;
    const uint32_t ncells = (uint32_t)((int64_t)G.nx * G.ny * G.nz);
    out->R = G;
    if (n == 0) return CUTE_OK;
    // regions on the device
    const int32_t* dreg = region;
    if (!regions_on_device) {
        int32_t* r = nullptr;
        if ((s = tmp.alloc(&r, (size_t)n)) != CUTE_OK) return s;
        CUTE_HIP(hipMemcpyAsync(r, region, (size_t)n * sizeof(int32_t), hipMemcpyHostToDevice, hs));
        dreg = r;
    }
    // the grid copy: same cells, the points of each cell sorted by region
    GridHost& R = out->R;
    unsigned char* blk = nullptr;
    const size_t b64 = (size_t)n * sizeof(P64), b32 = (size_t)n * sizeof(float4);
    if ((s = tmp.alloc(&blk, b64 + b32 + (size_t)n * (sizeof(uint32_t) + sizeof(uint16_t)))) != CUTE_OK) return s;
    R.block = blk;
    R.p64 = reinterpret_cast<P64*>(blk);
    R.p32 = reinterpret_cast<float4*>(blk + b64);
    out->rc = reinterpret_cast<uint32_t*>(blk + b64 + b32);
    out->regs = reinterpret_cast<uint16_t*>(out->rc + n);
    if ((s = tmp.alloc(&out->bad, 1)) != CUTE_OK) return s;
    if ((s = zero_u32(out->bad, 1, hs)) != CUTE_OK) return s;
    return (uint64_t)ncells * (uint64_t)K < (uint64_t(1) << 32)
               ? region_sort<uint32_t>(G, dreg, ncells, K, hs, tmp, out)
               : region_sort<uint64_t>(G, dreg, ncells, K, hs, tmp, out);
}

// One region pass: the region-pure home tiles of `home` against the
// neighbours of `nb` (the full stencil). Item k collects the pairs of the
// region-k home tiles, each weighted wsame when its neighbour's region
// (nb_regs) is k and wdiff otherwise (weight 1 without nb_regs); with h2, the
// 64-bit counters hold a pair of 32-bit ones (weights 1 and 1 << 32), and the
// sums of their high halves go there. selfx when home and neighbours are one
// catalog (pairs j != i in the home tile's own span). h (and h2) receive K
// histograms of nbins; st accumulates the statistics.
cute_status region_pass(const RegionCopy& home, const GridHost& nb, const uint16_t* nb_regs,
                        bool selfx, uint64_t wsame, uint64_t wdiff, int32_t K,
                        const cute_binning* bins, cute_precision prec, hipStream_t hs,
                        std::vector<uint64_t>* h, std::vector<uint64_t>* h2, cute_count_stats* st) {
    cute_status s;
    const GridHost& R = home.R;
    Plan pl;
    plan_binning(bins, pl);
    ItemGeom geo;
    if ((s = plan_item(R, nb, false, bins, pl, &geo)) != CUTE_OK) return s;
    if (selfx && geo.stencil.empty() && R.n > 0)
        return fail(CUTE_E_UNSUPPORTED, "stencil too large for the region pass");
    int kprec = plan_form(bins, geo.em, (int)prec, pl);
    if ((s = plan_lds(pl, 16, &kprec)) != CUTE_OK) return s;
    const size_t nbins = (size_t)pl.a.nbins, nh = (size_t)K * nbins;
    h->assign(nh, 0);
    if (h2) h2->assign(nh, 0);
    if (R.n == 0 || nb.n == 0) return CUTE_OK;
    int dev = 0, per_cu = 1, ncu = 0;
    if ((s = ensure_device_ready(&dev)) != CUTE_OK) return s;
    if ((s = batch_prepare(pl.mode, kprec, pl.est, pl.lds, &per_cu)) != CUTE_OK) return s;
    CUTE_HIP(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
    TempList tmp(hs);
    // how many home tiles each region has (one wait, which also brings the
    // verdict on the labels)
    uint32_t* doff = nullptr;   // offsets (K + 1) | fill counts (K)
    if ((s = tmp.alloc(&doff, 2 * (size_t)K + 1)) != CUTE_OK) return s;
    if ((s = region_tiles(R, geo.max_w, home.rc, (uint32_t)K, doff, nullptr, nullptr, hs)) != CUTE_OK) return s;
    std::vector<uint32_t> off((size_t)K + 1, 0);
    uint32_t bad = 0;
    CUTE_HIP(hipMemcpyAsync(off.data(), doff, off.size() * 4, hipMemcpyDeviceToHost, hs));
    CUTE_HIP(hipMemcpyAsync(&bad, home.bad, sizeof(bad), hipMemcpyDeviceToHost, hs));
    CUTE_HIP(hipStreamSynchronize(hs));
    if (bad) return fail(CUTE_E_INVALID_ARG, "region labels must be in [0, K)");
    const uint32_t ntiles = off[(size_t)K];
    Tile* dtiles = nullptr;
    if ((s = tmp.alloc(&dtiles, std::max<size_t>(ntiles, 1))) != CUTE_OK) return s;
    if ((s = region_tiles(R, geo.max_w, home.rc, (uint32_t)K, doff, doff + K + 1, dtiles, hs)) != CUTE_OK) return s;
    // the regions that have tiles, the workgroups shared out by their tiles
    // (half the tiles: twelve tasks per slot, since a region's workgroups wait
    // for their last tasks at every change of region; three, six and twelve take
    // 4.30, 3.75 and 3.51 ms per jackknife of 2.5e5 points in 100 regions)
    const int plog = part_log(0.5 * (double)ntiles, geo.near, ncu);
    const int gsz = (int)std::min<uint64_t>((uint64_t)per_cu * ncu,
                                            (((uint64_t)ntiles << plog) + kWgWaves - 1) / kWgWaves);
    std::vector<uint32_t> nt(2 * (size_t)K), lst, first;
    std::vector<double> share;
    for (int k = 0; k < K; k++) {
        nt[2 * (size_t)k] = off[k + 1] - off[k];
        nt[2 * (size_t)k + 1] = (uint32_t)plog;
        if (nt[2 * (size_t)k] == 0) continue;
        lst.push_back((uint32_t)k);
        share.push_back((double)nt[2 * (size_t)k]);
    }
    if (!lst.empty()) first = batch_first(share, gsz);
    // device block of the launch, filled by one copy:
    // [T1 | T2 | B1 | B2 | stencil | tiles and parts per region | list | first | args]
    std::vector<unsigned char> img;
    auto put = [&](const void* p, size_t bytes) {
        const size_t o = img.size();
        img.resize(o + ((bytes + 15) & ~(size_t)15));
        if (bytes) memcpy(img.data() + o, p, bytes);
        return o;
    };
    const size_t oT1 = put(pl.T1.data(), pl.T1.size() * 8), oT2 = put(pl.T2.data(), pl.T2.size() * 8);
    const size_t oB1 = put(pl.band1.data(), pl.band1.size() * 8), oB2 = put(pl.band2.data(), pl.band2.size() * 8);
    const size_t oST = put(geo.stencil.data(), geo.stencil.size() * sizeof(int4));
    const size_t oNT = put(nt.data(), nt.size() * 4), oLS = put(lst.data(), lst.size() * 4);
    const size_t oFI = put(first.data(), first.size() * 4);
    const size_t oAR = img.size(), total = oAR + sizeof(CountArgs) * (size_t)K;
    unsigned char* blob = nullptr;
    unsigned long long* work = nullptr;  // K * nbins histograms (twice with h2), 4 stats and a head per item, done
    const size_t hists = h2 ? 2 * nh : nh, wwords = hists + 5 * (size_t)K + 1;
    if ((s = tmp.alloc(&blob, total)) != CUTE_OK) return s;
    if ((s = tmp.alloc(&work, wwords)) != CUTE_OK) return s;
    if ((s = zero_u64(work, wwords, hs)) != CUTE_OK) return s;
    CountArgs* dargs = reinterpret_cast<CountArgs*>(blob + oAR);
    img.resize(total);
    for (int k = 0; k < K; k++) {
        CountArgs a = pl.a;
        apply_item(geo, &a);
        a.self = dargs + k;
        a.T1 = reinterpret_cast<const double*>(blob + oT1);
        a.T2 = reinterpret_cast<const double*>(blob + oT2);
        a.band1 = reinterpret_cast<const float2*>(blob + oB1);
        a.band2 = reinterpret_cast<const float2*>(blob + oB2);
        a.stencil = geo.stencil.empty() ? nullptr : reinterpret_cast<const int4*>(blob + oST);
        a.nst = (int)geo.stencil.size();
        a.tiles = dtiles + off[k];
        a.ntiles = nt[2 * (size_t)k];
        a.counts = work + (size_t)k * nbins;
        a.counts_hi = h2 ? work + nh + (size_t)k * nbins : nullptr;
        a.stats = work + hists + 4 * (size_t)k;
        a.regs = nb_regs;
        a.region = k;
        a.wsame = wsame;
        a.wdiff = wdiff;
        a.selfx = selfx ? 1 : 0;
        memcpy(img.data() + oAR + sizeof(CountArgs) * (size_t)k, &a, sizeof(a));
    }
    CUTE_HIP(hipMemcpyAsync(blob, img.data(), total, hipMemcpyHostToDevice, hs));
    BatchArgs ba;
    memset(&ba, 0, sizeof(ba));
    ba.items = dargs;
    ba.list = reinterpret_cast<const uint32_t*>(blob + oLS);
    ba.nlist = (uint32_t)lst.size();
    ba.first = reinterpret_cast<const uint32_t*>(blob + oFI);
    ba.ntiles = reinterpret_cast<const uint32_t*>(blob + oNT);
    ba.heads = work + hists + 4 * (size_t)K;
    ba.done = ba.heads + K;
    ba.n1 = pl.a.n1;
    ba.n2 = pl.a.n2;
    ba.nbins = pl.a.nbins;
    ba.copies = pl.a.copies;
    ba.hist_words = pl.a.hist_words;
    ba.T1 = reinterpret_cast<const double*>(blob + oT1);
    ba.T2 = reinterpret_cast<const double*>(blob + oT2);
    ba.band1 = reinterpret_cast<const float2*>(blob + oB1);
    ba.band2 = reinterpret_cast<const float2*>(blob + oB2);
    double ms = 0.0;
    if (ntiles) {
        EventTimer timer(hs);
        if ((s = batch_launch(ba, pl.mode, kprec, pl.est, gsz, pl.lds, hs)) != CUTE_OK) return s;
        timer.stop();
        ms = timer.elapsed_ms();
    }
    // the histograms come back through pinned memory unless they are large
    HostStage stage(hs);
    std::vector<unsigned char> pageable;
    unsigned char* hb = nullptr;
    if (wwords * 8 > ((size_t)8 << 20)) {
        pageable.resize(wwords * 8);
        hb = pageable.data();
    } else if ((s = stage.get(wwords * 8, &hb)) != CUTE_OK) {
        return s;
    }
    CUTE_HIP(hipMemcpyAsync(hb, work, wwords * 8, hipMemcpyDeviceToHost, hs));
    CUTE_HIP(hipStreamSynchronize(hs));
    const unsigned long long* hw = reinterpret_cast<const unsigned long long*>(hb);
    uint64_t tiles_done = 0;
    for (int k = 0; k < K; k++) {
        const unsigned long long* sv = hw + hists + 4 * (size_t)k;
        st->pair_evals += sv[0];
        st->retests += sv[1];
        st->flips += sv[2];
        tiles_done += sv[3];
    }
    st->tiles += tiles_done;
    st->ms_count += ms;
    if (tiles_done != ntiles) return fail(CUTE_E_INTERNAL, "not every region tile was processed");
    for (size_t i = 0; i < nh; i++) (*h)[i] = hw[i];
    if (h2)
        for (size_t i = 0; i < nh; i++) (*h2)[i] = hw[nh + i];
    return CUTE_OK;
}

cute_status check_common(const cute_grid* g, const int32_t* region, int32_t K,
                         const cute_binning* bins, cute_precision prec) {
    // every argument is checked before the grid is read
    if (!g || !region) return fail(CUTE_E_INVALID_ARG, "NULL argument");
    if (K < 1 || K > 65535) return fail(CUTE_E_INVALID_ARG, "K must be in [1, 65535]");
    cute_status s = validate_binning(bins);
    if (s != CUTE_OK) return s;
    if (prec != CUTE_PREC_FP64 && prec != CUTE_PREC_FP32_EDGE && prec != CUTE_PREC_FP32_ONLY)
        return fail(CUTE_E_INVALID_ARG, "unknown precision");
    if (g->h.wt != nullptr) return fail(CUTE_E_UNSUPPORTED, "pixel maps have no jackknife pass");
    if (g->h.geom == CUTE_GEOM_SPHERE) return fail(CUTE_E_UNSUPPORTED, "jackknife regions need a 3-D grid");
    return CUTE_OK;
}

// whether a jackknife's region pass also gives its total (64-bit counters, and
// decisions that do not depend on which point of a pair is the home)
bool one_pass(const cute_binning* b, cute_precision prec) {
    const bool mid = b->kind == CUTE_BIN_SIGMAPI || (b->kind == CUTE_BIN_RMU && b->los == CUTE_LOS_MIDPOINT);
    return !mid && prec != CUTE_PREC_FP32_ONLY;
}

void add_stats(cute_count_stats* st, const cute_count_stats& a, const cute_count_stats& b) {
    if (!st) return;
    *st = a;
    st->pair_evals += b.pair_evals;
    st->retests += b.retests;
    st->flips += b.flips;
    st->tiles += b.tiles;
    st->ms_count += b.ms_count;
}

}  // namespace

extern "C" cute_status cute_count_jackknife(const cute_grid* grid, const int32_t* region,
                                            int32_t regions_on_device, int32_t K,
                                            const cute_binning* bins, cute_precision prec,
                                            uint64_t* total, uint64_t* jack,
                                            cute_count_stats* st, void* stream) {
    if (!total || !jack) return fail(CUTE_E_INVALID_ARG, "NULL argument");
    cute_status s = check_common(grid, region, K, bins, prec);
    if (s != CUTE_OK) return s;
    const GridHost& G = grid->h;
    hipStream_t hs = (hipStream_t)stream;
    cute_count_stats st_tot, st_reg;
    memset(&st_tot, 0, sizeof(st_tot));
    memset(&st_reg, 0, sizeof(st_reg));
    const int nbins = bins->n1 * (bins->n2 > 0 ? bins->n2 : 1);
    const bool both = one_pass(bins, prec) && G.n > 0;
    if (!both && (s = cute_count_pairs(grid, nullptr, bins, prec, total, 0, &st_tot, stream)) != CUTE_OK)
        return s;
    std::vector<uint64_t> h1((size_t)K * nbins, 0), h2;
    if (G.n > 0) {
        if (both && (s = grid_wait(grid, hs)) != CUTE_OK) return s;
        TempList tmp(hs);
        RegionCopy rc;
        if ((s = region_copy(G, region, regions_on_device, K, hs, tmp, &rc)) != CUTE_OK) return s;
        if ((s = region_pass(rc, rc.R, rc.regs, true, 1u, both ? uint64_t(1) << 32 : 2u, K, bins, prec, hs, &h1,
                             both ? &h2 : nullptr, &st_reg)) != CUTE_OK)
            return s;
    }
    if (both) {
        for (int b = 0; b < nbins; b++) {
            uint64_t t = 0;
            for (int k = 0; k < K; k++) t += h1[(size_t)k * nbins + b] + h2[(size_t)k * nbins + b];
            if (t & 1u) return fail(CUTE_E_INTERNAL, "region histograms are inconsistent");
            total[b] = t / 2;
            st_tot.pairs_in_range += total[b];
        }
    }
    // jack_k = total - T_k
    for (int k = 0; k < K; k++)
        for (int b = 0; b < nbins; b++) {
            const uint64_t w = h1[(size_t)k * nbins + b];
            const uint64_t t = w / 2 + (both ? h2[(size_t)k * nbins + b] : 0);
            if ((w & 1u) || t > total[b])
                return fail(CUTE_E_INTERNAL, "region histograms are inconsistent");
            jack[(size_t)k * nbins + b] = total[b] - t;
        }
    add_stats(st, st_tot, st_reg);
    return CUTE_OK;
}

extern "C" cute_status cute_count_jackknife_cross(const cute_grid* a, const int32_t* region_a,
                                                  const cute_grid* b, const int32_t* region_b,
                                                  int32_t regions_on_device, int32_t K,
                                                  const cute_binning* bins, cute_precision prec,
                                                  uint64_t* total, uint64_t* jack,
                                                  cute_count_stats* st, void* stream) {
    if (!total || !jack || !a || !region_a || !b || !region_b)
        return fail(CUTE_E_INVALID_ARG, "NULL argument");
    if (K < 1 || K > 65535) return fail(CUTE_E_INVALID_ARG, "K must be in [1, 65535]");
    cute_status s = check_common(a, region_a, K, bins, prec);
    if (s != CUTE_OK) return s;
    if ((s = check_common(b, region_b, K, bins, prec)) != CUTE_OK) return s;
    if (a == b) return fail(CUTE_E_INVALID_ARG, "a and b are one grid: use cute_count_jackknife");
    hipStream_t hs = (hipStream_t)stream;
    cute_count_stats st_tot, st_reg;
    memset(&st_tot, 0, sizeof(st_tot));
    memset(&st_reg, 0, sizeof(st_reg));
    const int nbins = bins->n1 * (bins->n2 > 0 ? bins->n2 : 1);
    const bool sum = prec != CUTE_PREC_FP32_ONLY && a->h.n > 0 && b->h.n > 0;
    if (!sum && (s = cute_count_pairs(a, b, bins, prec, total, 0, &st_tot, stream)) != CUTE_OK) return s;
    std::vector<uint64_t> ha((size_t)K * nbins, 0), hb((size_t)K * nbins, 0);
    if (a->h.n > 0 && b->h.n > 0) {
        if (sum && (s = grid_wait(a, hs)) != CUTE_OK) return s;
        if (sum && (s = grid_wait(b, hs)) != CUTE_OK) return s;
        TempList tmp(hs);
        RegionCopy ra, rb;
        if ((s = region_copy(a->h, region_a, regions_on_device, K, hs, tmp, &ra)) != CUTE_OK) return s;
        if ((s = region_copy(b->h, region_b, regions_on_device, K, hs, tmp, &rb)) != CUTE_OK) return s;
        // pairs whose A point lies in region k
        if ((s = region_pass(ra, b->h, nullptr, false, 1u, 1u, K, bins, prec, hs, &ha, nullptr,
                             &st_reg)) != CUTE_OK)
            return s;
        // pairs whose B point lies in region k and whose A point does not
        if ((s = region_pass(rb, ra.R, ra.regs, false, 0u, 1u, K, bins, prec, hs, &hb, nullptr,
                             &st_reg)) != CUTE_OK)
            return s;
    }
    if (sum) {
        for (int c = 0; c < nbins; c++) {
            total[c] = 0;
            for (int k = 0; k < K; k++) total[c] += ha[(size_t)k * nbins + c];
            st_tot.pairs_in_range += total[c];
        }
    }
    for (int k = 0; k < K; k++)
        for (int c = 0; c < nbins; c++) {
            const size_t i = (size_t)k * nbins + c;
            const uint64_t t = ha[i] + hb[i];
            if (t > total[c]) return fail(CUTE_E_INTERNAL, "region histograms are inconsistent");
            jack[i] = total[c] - t;
        }
    add_stats(st, st_tot, st_reg);
    return CUTE_OK;
}
