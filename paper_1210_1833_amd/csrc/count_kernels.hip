// Pair-count kernels for gfx950.
//
// One wavefront owns one home tile at a time (a run of up to 64 sorted points
// inside one row of cells) and walks the neighbour cells of Sec. 3.3 as
// contiguous spans of the other catalog. The spans are cut into chunks of 64
// neighbour points, one per lane in VGPRs. A step evaluates four home points
// against them, four independent pairs per lane: in FP32_EDGE the separations
// are matrix products whose rows are home points staged in LDS (or, where that
// form would re-test too many pairs, differences of components, see
// plan_form); there and in the other paths the home points are wave-uniform
// and arrive through scalar loads. Counts go to one LDS histogram per
// workgroup (several interleaved copies, so that lanes hitting the same bin
// use different banks; 64-bit counters, 32-bit ones for the midpoint kinds),
// summed into uint64 global counts at the end.
//
// Precision paths
//  - FP64: every pair is classified by the canonical FP64 predicates.
//  - FP32_EDGE: separations in FP32; a pair is counted directly only when its
//    FP32 value is farther than a proven rounding bound from every decision
//    threshold (bin edges, r_max, mu edges); the rest go to a per-wave LDS
//    queue that is drained 64 pairs at a time through the canonical FP64
//    predicates, so the counts equal the FP64 ones.
//  - FP32_ONLY: FP32 decisions only.
#include <map>
#include <mutex>
#include <tuple>

#include "count_device.h"

namespace cute {

namespace {

// Four 4-wave workgroups per CU: the register budget stays at 128 VGPRs.
// The FP32_EDGE kernels without a pair line of sight run five (96 VGPRs),
// which hides more latency: the angular count took 10 % less time, the region
// pass of 1500 bins 4 %; the midpoint kinds would spill.
// WT: pixel maps, each pair weighted by the product of the point weights.
template <int MODE, int PREC, int EST, bool WT>
__global__ __launch_bounds__(256, (kWgPerCu<MODE, PREC>)) void k_count(CountArgs P) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int nwaves = blockDim.x >> 6;
    const int n1 = P.n1;
    const int n2p = P.n2 > 0 ? P.n2 : 0;
    constexpr bool H32 = kH32<MODE>;
    const WgLds L = wg_lds<H32, kMfma<MODE, PREC, EST>, kAlpha<MODE>>(smem, nwaves, n1, P.n2, P.hist_words);
    double *T1 = L.T1, *T2 = L.T2;
    float2 *B1 = L.B1, *B2 = L.B2;
    unsigned char* hist0 = L.hist;
    for (int i = threadIdx.x; i <= n1; i += blockDim.x) T1[i] = P.T1[i];
    for (int i = threadIdx.x; i <= n2p; i += blockDim.x) T2[i] = n2p ? P.T2[i] : 0.0;
    if (PREC != P_FP64) {
        // (sigma-pi from the matrix cores: one entry past the last bin)
        constexpr int more = kMfma<MODE, PREC, EST> && MODE == M_SIGMAPI ? 1 : 0;
        for (int i = threadIdx.x; i < n1 + more; i += blockDim.x) B1[i] = P.band1[i];
        for (int i = threadIdx.x; i < n2p + more; i += blockDim.x) B2[i] = P.band2[i];
    }
    for (size_t i = threadIdx.x; i < L.hbytes / 4; i += blockDim.x) reinterpret_cast<uint32_t*>(hist0)[i] = 0u;
    for (int i = threadIdx.x; i < 2 * nwaves; i += blockDim.x) L.rstat[i] = 0ull;
    if (H32 && threadIdx.x == 0) L.ctl[0] = 0u;
    __syncthreads();

    WaveState W = wave_state(L, wave);
    W.budget = L.ctl;   // 32-bit histograms only
    SpanBuf S = span_buf(L, wave);

    // tasks: the parts of the tiles (see part_rule). Every wave starts with the task of its
    // own number, so that a launch of no more tasks than waves pops none; an
    // empty tile slot is no tile.
    const uint32_t plog = P.ntiles_dev ? uni(P.ntiles_dev[1]) : (uint32_t)P.plog;
    const uint32_t ntasks = (P.ntiles_dev ? uni(P.ntiles_dev[0]) : P.ntiles) << plog;
    const uint32_t nw = gridDim.x * (uint32_t)nwaves;
    for (uint32_t t = blockIdx.x * (uint32_t)nwaves + (uint32_t)unii(wave); t < ntasks;) {
        const cu32p tp = (cu32p)(const void*)P.tiles + 4 * (size_t)(t >> plog);
        Tile tl;
        tl.start = uni(tp[0]);
        tl.end = uni(tp[1]);
        tl.row = uni(tp[2]);
        tl.c0c1 = uni(tp[3]);
        if (tl.end > tl.start)
            do_tile<MODE, PREC, EST, false, WT>(P, W, S, B1, B2, T1, T2, lane, tl,
                                                t & ((1u << plog) - 1u), plog);
        if (ntasks <= nw) break;
        uint32_t nx = 0;
        if (lane == 0) nx = atomicAdd(P.work_head, 1u);
        t = nw + uni(nx);
    }
    if constexpr (PREC == P_FP32E)
        W.tail = drain_queue<MODE, EST>(P.self, W.hist, W.qi, W.qj, W.qc, W.rstat, B1, B2, T1, T2, lane,
                                        W.tail, true);
    // the statistics of the four waves, through their (empty) queues, in one
    // atomic instruction: four per wave, to one line, were 20 000 at the end of
    // a full launch (FP64 r-mu count of 4e5 points: 1.82 ms, 1.62 so)
    unsigned long long* wst = reinterpret_cast<unsigned long long*>(W.qi);
    if (lane == 0) {
        wst[0] = W.evals;
        wst[1] = W.rstat[0];
        wst[2] = W.rstat[1];
        wst[3] = W.tiles;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        unsigned long long t = 0;
        for (int w = 0; w < nwaves; w++)
            t += reinterpret_cast<const unsigned long long*>(L.queue + (size_t)w * 2 * kQCap)[threadIdx.x];
        atomicAdd(&P.stats[threadIdx.x], t);
    }
    // sum the copies, then one global atomic per non-empty bin
    for (int b = threadIdx.x; b < P.nbins; b += blockDim.x) {
        uint64_t s = 0;
        if constexpr (H32) {
            const uint32_t* hh = reinterpret_cast<const uint32_t*>(hist0) + (size_t)b * P.copies;
            for (int c = 0; c < P.copies; c++) s += hh[c];
        } else {
            const unsigned long long* hh = reinterpret_cast<const unsigned long long*>(hist0) + (size_t)b * P.copies;
            for (int c = 0; c < P.copies; c++) s += hh[c];
        }
        if (s) atomicAdd(&P.counts[b], (unsigned long long)s);
    }
}

template <int MODE, int PREC, int EST, bool WT>
cute_status launch_one(const CountArgs& a, int wg_waves, size_t lds, hipStream_t s, int* grid_used) {
    auto kern = k_count<MODE, PREC, EST, WT>;
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void*)kern,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return hip_status(e, "hipFuncSetAttribute");
    }
    // occupancy of this variant at this LDS size, queried once per device
    static std::mutex mu;
    static std::map<std::tuple<int, int, size_t, bool>, std::pair<int, int>> cache;
    int dev = 0, ncu = 0, per_cu = 0;
    CUTE_HIP(hipGetDevice(&dev));
    {
        std::lock_guard<std::mutex> lk(mu);
        auto it = cache.find(std::make_tuple(dev, wg_waves, lds, WT));
        if (it != cache.end()) {
            ncu = it->second.first;
            per_cu = it->second.second;
        }
    }
    if (ncu == 0) {
        CUTE_HIP(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
        CUTE_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kern, 64 * wg_waves, lds));
        if (per_cu < 1) per_cu = 1;
        std::lock_guard<std::mutex> lk(mu);
        cache[std::make_tuple(dev, wg_waves, lds, WT)] = std::make_pair(ncu, per_cu);
    }
    int64_t want = (int64_t)per_cu * ncu;
    if (a.tiles == nullptr) {   // only asked how many workgroups run at a time
        if (grid_used) *grid_used = (int)want;
        return CUTE_OK;
    }
    int64_t need = (((int64_t)a.ntiles << a.plog) + wg_waves - 1) / wg_waves;
    int grid = (int)(want < need ? want : need);
    if (grid < 1) grid = 1;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(64 * wg_waves), lds, s, a);
    CUTE_HIP(hipGetLastError());
    if (grid_used) *grid_used = grid;
    return CUTE_OK;
}

template <int MODE, int PREC>
cute_status launch_est(const CountArgs& a, int est, int wg_waves, size_t lds, hipStream_t s,
                       int* g) {
    if (a.wA != nullptr) {
        // weighted pairs: the angular kernels only (pixel maps)
        if constexpr (MODE == M_THETA) {
            if constexpr (PREC == P_FP32E) {
                if (est == (E_DIF | E_LOG)) return launch_one<MODE, PREC, E_DIF | E_LOG, true>(a, wg_waves, lds, s, g);
                if (est == E_DIF) return launch_one<MODE, PREC, E_DIF, true>(a, wg_waves, lds, s, g);
            }
            if (est_log(est)) return launch_one<MODE, PREC, E_LOG, true>(a, wg_waves, lds, s, g);
            return launch_one<MODE, PREC, E_LIN, true>(a, wg_waves, lds, s, g);
        } else {
            return fail(CUTE_E_UNSUPPORTED, "weighted pairs need a THETA binning");
        }
    }
    if constexpr (PREC == P_FP32E) {
        // component-wise separations, and the mu decision in mu space
        if constexpr (MODE == M_RMU_Z) {
            if (est == (E_DIF | E_LOG | E_MUF))
                return launch_one<MODE, PREC, E_DIF | E_LOG | E_MUF, false>(a, wg_waves, lds, s, g);
            if (est == (E_DIF | E_MUF)) return launch_one<MODE, PREC, E_DIF | E_MUF, false>(a, wg_waves, lds, s, g);
        }
        if constexpr (MODE != M_SIGMAPI)
            if (est == (E_DIF | E_LOG)) return launch_one<MODE, PREC, E_DIF | E_LOG, false>(a, wg_waves, lds, s, g);
        if (est == E_DIF) return launch_one<MODE, PREC, E_DIF, false>(a, wg_waves, lds, s, g);
        if constexpr (MODE == M_RMU_Z || MODE == M_RMU_MID) {
            if (est == (E_LOG | E_MUF)) return launch_one<MODE, PREC, E_LOG | E_MUF, false>(a, wg_waves, lds, s, g);
            if (est == E_MUF) return launch_one<MODE, PREC, E_MUF, false>(a, wg_waves, lds, s, g);
        }
        if constexpr (MODE == M_RMU_Z || MODE == M_RMU_MID) return fail(CUTE_E_INTERNAL, "unknown kernel variant");
    }
    constexpr bool general = PREC != P_FP32E || (MODE != M_RMU_Z && MODE != M_RMU_MID);
    if constexpr (general && MODE != M_SIGMAPI)   // (sigma is estimated linearly)
        if (est_log(est)) return launch_one<MODE, PREC, E_LOG, false>(a, wg_waves, lds, s, g);
    if constexpr (general) return launch_one<MODE, PREC, E_LIN, false>(a, wg_waves, lds, s, g);
}

template <int MODE>
cute_status launch_prec(const CountArgs& a, int prec, int est, int wg_waves, size_t lds,
                        hipStream_t s, int* g) {
    switch (prec) {
        case P_FP64: return launch_est<MODE, P_FP64>(a, est, wg_waves, lds, s, g);
        case P_FP32E: return launch_est<MODE, P_FP32E>(a, est, wg_waves, lds, s, g);
        default: return launch_est<MODE, P_FP32O>(a, est, wg_waves, lds, s, g);
    }
}

}  // namespace

cute_status launch_count(const CountArgs& args, int mode, int prec, int est, int wg_waves,
                         size_t lds_bytes, hipStream_t stream, int* grid_used) {
    switch (mode) {
        case M_MONO: return launch_prec<M_MONO>(args, prec, est, wg_waves, lds_bytes, stream, grid_used);
        case M_RMU_Z: return launch_prec<M_RMU_Z>(args, prec, est, wg_waves, lds_bytes, stream, grid_used);
        case M_RMU_MID: return launch_prec<M_RMU_MID>(args, prec, est, wg_waves, lds_bytes, stream, grid_used);
        case M_SIGMAPI: return launch_prec<M_SIGMAPI>(args, prec, est, wg_waves, lds_bytes, stream, grid_used);
        case M_THETA: return launch_prec<M_THETA>(args, prec, est, wg_waves, lds_bytes, stream, grid_used);
        case M_RADIAL:
            if (prec == P_FP32O || args.wA != nullptr)
                return fail(CUTE_E_UNSUPPORTED, "radial counts are exact and unweighted");
            if (prec == P_FP32E)
                return launch_one<M_RADIAL, P_FP32E, E_LIN, false>(args, wg_waves, lds_bytes, stream, grid_used);
            return launch_one<M_RADIAL, P_FP64, E_LIN, false>(args, wg_waves, lds_bytes, stream, grid_used);
        default: return fail(CUTE_E_INTERNAL, "unknown mode");
    }
}

// Home tiles: each row of cells is cut into runs of at most tmax points
// whose x-extent stays within max_w cells (so that periodic stencils never
// wrap onto themselves); a cell with more points is split. One thread walks
// one row; with out == nullptr it only counts the tiles.
__device__ uint32_t walk_row_tiles(const uint32_t* __restrict__ cstart, int nx, int r, int max_w,
                                   uint32_t tmax, Tile* __restrict__ out) {
    const uint32_t* cs = cstart + (size_t)r * nx;
    uint32_t o = 0, fill = 0;
    int first = -1;
    Tile cur{0u, 0u, 0u, 0u};
    bool open = false;
    // cell offsets in batches of eight (independent loads in flight); the
    // batch loop is unrolled so that the offsets stay in registers
    constexpr int kB = 8;
    for (int cb = 0; cb < nx; cb += kB) {
        uint32_t ofs[kB + 1];
#pragma unroll
        for (int i = 0; i <= kB; i++) ofs[i] = cb + i <= nx ? cs[cb + i] : 0u;
#pragma unroll
        for (int k = 0; k < kB; k++) {
            const int c = cb + k;
            if (c >= nx) break;
            uint32_t pos = ofs[k];
            const uint32_t end = ofs[k + 1];
            while (pos < end) {
                if (!open || fill == tmax || c - first + 1 > max_w) {
                    if (open) {
                        if (out) out[o] = cur;
                        o++;
                    }
                    open = true;
                    fill = 0;
                    first = c;
                    cur.start = pos;
                    cur.end = pos;
                    cur.row = (uint32_t)r;
                    cur.c0c1 = (uint32_t)c | ((uint32_t)c << 16);
                }
                const uint32_t take = tmax - fill < end - pos ? tmax - fill : end - pos;
                fill += take;
                pos += take;
                cur.end = pos;
                cur.c0c1 = (cur.c0c1 & 0xffffu) | ((uint32_t)c << 16);
            }
        }
    }
    if (open) {
        if (out) out[o] = cur;
        o++;
    }
    return o;
}

__global__ __launch_bounds__(256) void k_tiles_count(const uint32_t* __restrict__ cstart,
                                                     int nx, int nrows, int max_w, uint32_t tmax,
                                                     uint32_t* __restrict__ ntile) {
    int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r == 0) ntile[nrows] = 0u;  // the scan's last entry becomes the total
    if (r >= nrows) return;
    ntile[r] = walk_row_tiles(cstart, nx, r, max_w, tmax, nullptr);
}

__global__ __launch_bounds__(256) void k_tiles_write(const uint32_t* __restrict__ cstart,
                                                     int nx, int nrows, int max_w, uint32_t tmax,
                                                     const uint32_t* __restrict__ toff,
                                                     Tile* __restrict__ tiles,
                                                     uint32_t* __restrict__ total) {
    int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r == 0 && total != nullptr) *total = toff[nrows];
    if (r >= nrows) return;
    (void)walk_row_tiles(cstart, nx, r, max_w, tmax, tiles + toff[r]);
}

// Region tiles (see region_tiles), one wave per row: a tile is the run of
// points from its first on, up to tmax, in its region and within max_w cells of
// its first cell, found by one vote of the lanes, which hold 64 points; a run
// that reaches the last of them is looked at again from its own first point.
// The tiles of one region are kept in the lanes and reserved with one atomic
// (one per tile made the pass wait for the few counters: 80 us for 2.5e5 points
// in 100 regions; a walk of single points by one thread per row took 590). The
// first pass counts the tiles of each region, the second writes them, in any
// order within their region.
template <bool WRITE>
__global__ __launch_bounds__(256) void k_region_tiles(const uint32_t* __restrict__ cstart, int nx, int nrows,
                                                      int max_w, uint32_t tmax,
                                                      const uint32_t* __restrict__ rc,
                                                      uint32_t* __restrict__ cnt,
                                                      const uint32_t* __restrict__ off,
                                                      Tile* __restrict__ out) {
    const int lane = (int)(threadIdx.x & 63u);
    const int r = unii((int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6));
    if (r >= nrows) return;
    const uint32_t* cs = cstart + (size_t)r * nx;
    const uint32_t p1 = uni(cs[nx]);
    // the tiles of region cr not written yet, tile k in lane k
    uint32_t m = 0, cr = 0;
    Tile tl{0u, 0u, 0u, 0u};
    auto flush = [&]() {
        uint32_t k = 0;
        if (lane == 0) k = atomicAdd(&cnt[cr], m);
        if (WRITE) {
            k = uni(k) + off[cr] + (uint32_t)lane;
            if ((uint32_t)lane < m) out[k] = tl;
        }
        m = 0;
    };
    for (uint32_t p = uni(cs[0]); p < p1;) {
        const uint32_t n = p1 - p < 64u ? p1 - p : 64u;
        const uint32_t v = (uint32_t)lane < n ? rc[p + (uint32_t)lane] : 0u;
        uint32_t o = 0;
        do {
            // the run from point p + o on (lane o is in it)
            const uint32_t v0 = lane_u32(v, (int)o), rg = v0 >> 16, c0 = v0 & 0xffffu;
            const bool in = (uint32_t)lane - o < tmax && (uint32_t)lane < n && (v >> 16) == rg &&
                            (v & 0xffffu) - c0 < (uint32_t)max_w;
            const uint64_t no = ~__builtin_amdgcn_ballot_w64(in) >> o;
            const uint32_t len = no != 0ull ? (uint32_t)__builtin_ctzll(no) : 64u - o;
            if (o + len >= 64u && o > 0u) break;
            const uint32_t c1 = lane_u32(v, (int)(o + len) - 1) & 0xffffu;
            if (m == 64u || (m != 0u && rg != cr)) flush();
            cr = rg;
            if ((uint32_t)lane == m) tl = Tile{p + o, p + o + len, (uint32_t)r, c0 | (c1 << 16)};
            m++;
            o += len;
        } while (o < n);
        p += o;
    }
    if (m != 0u) flush();
}

// Tiles without a count pass. Row r, whose points are [s_r, s_{r+1}), owns
// the slots from b_r = floor(s_r / tmax) + r (W + 1), W = floor((nx - 1) /
// max_w), up to b_{r+1}: the rows partition [0, tile_count_bound) exactly, so
// every slot is written, with a tile or as empty. A row of p points has at
// most floor(p / tmax) + W + 1 tiles (see tile_count_bound), which is at most
// b_{r+1} - b_r because floor(s / tmax) + floor(p / tmax) <= floor((s + p) /
// tmax). The last row also takes any slots left before cap, the length of
// out, and no row writes at or past cap. A row with more tiles than slots
// (the bound failing) raises *overflow.
// One wave per row: the lanes load 64 cell offsets at a time, the walk (the
// cuts of walk_row_tiles without regions, on wave-uniform values) reads them
// with readlane, lane 0 writes the tiles and all lanes the empty slots.
__global__ __launch_bounds__(256) void k_tiles_sparse(const uint32_t* __restrict__ cstart, int nx,
                                                      int nrows, int max_w, uint32_t tmax,
                                                      Tile* __restrict__ out, uint32_t cap,
                                                      uint32_t* __restrict__ overflow,
                                                      uint32_t* __restrict__ total) {
    const int lane = (int)(threadIdx.x & 63u);
    const int r = unii((int)((blockIdx.x * blockDim.x + threadIdx.x) >> 6));
    if (r >= nrows) return;
    const uint32_t* cs = cstart + (size_t)r * nx;
    const uint64_t W1 = (uint64_t)((uint32_t)(nx - 1) / (uint32_t)max_w) + 1u;
    const uint32_t p0 = uni(cs[0]), p1 = uni(cs[nx]);
    const uint64_t b0 = (uint64_t)(p0 / tmax) + (uint64_t)r * W1;
    uint64_t b1 = r + 1 == nrows ? (uint64_t)cap : (uint64_t)(p1 / tmax) + (uint64_t)(r + 1) * W1;
    bool over = false;
    if (b1 > cap) {
        over = true;
        b1 = cap;
    }
    const uint32_t slots = b0 < b1 ? (uint32_t)(b1 - b0) : 0u;
    Tile* o = out + b0;
    uint32_t k = 0, fill = 0;
    int first = -1;
    bool open = false;
    Tile cur{0u, 0u, 0u, 0u};
    for (int cb = 0; cb < nx; cb += 64) {
        // offsets of cells cb .. cb + 63 in the lanes, of cell cb + 64 beside
        const uint32_t v = cb + lane <= nx ? cs[cb + lane] : 0u;
        const uint32_t vn = cb + 64 <= nx ? uni(cs[cb + 64]) : 0u;
        const int m = nx - cb < 64 ? nx - cb : 64;
        for (int j = 0; j < m; j++) {
            const int c = cb + j;
            uint32_t pos = (uint32_t)__builtin_amdgcn_readlane((int)v, j);
            const uint32_t end = j + 1 < 64 ? (uint32_t)__builtin_amdgcn_readlane((int)v, j + 1) : vn;
            while (pos < end) {
                if (!open || fill == tmax || c - first + 1 > max_w) {
                    if (open) {
                        if (lane == 0 && k < slots) o[k] = cur;
                        k++;
                    }
                    open = true;
                    fill = 0;
                    first = c;
                    cur.start = pos;
                    cur.end = pos;
                    cur.row = (uint32_t)r;
                    cur.c0c1 = (uint32_t)c | ((uint32_t)c << 16);
                }
                const uint32_t take = tmax - fill < end - pos ? tmax - fill : end - pos;
                fill += take;
                pos += take;
                cur.end = pos;
                cur.c0c1 = (cur.c0c1 & 0xffffu) | ((uint32_t)c << 16);
            }
        }
    }
    if (open) {
        if (lane == 0 && k < slots) o[k] = cur;
        k++;
    }
    if ((over || k > slots) && lane == 0) atomicOr(overflow, 1u);
    if (total != nullptr && k > 0u && lane == 0) atomicAdd(total, k);
    for (uint32_t i = k + (uint32_t)lane; i < slots; i += 64u) o[i] = Tile{0u, 0u, 0u, 0u};
}

namespace {

// Estimated cost of each home tile for the longest-first order: candidate
// pairs (home points times the neighbours its stencil rows hold) plus a
// per-row and a per-tile overhead, in pair evaluations.
constexpr uint32_t kCostBuckets = 256;

constexpr uint32_t kNoTile = 0xffffffffu;  // the key of an empty slot

// One wave per tile slot, the lanes taking the stencil rows; writes the
// tile's cost bucket to key[t] (kNoTile for an empty slot).
template <bool SPH>
__global__ __launch_bounds__(256) void k_tile_cost(CountArgs P, const Tile* __restrict__ tiles,
                                                   uint32_t ntiles, uint32_t* __restrict__ key) {
    const int lane = (int)(threadIdx.x & 63u);
    const uint32_t t = uni((blockIdx.x * blockDim.x + threadIdx.x) >> 6);
    if (t >= ntiles) return;
    const cu32p tp = (cu32p)(const void*)tiles;
    Tile tl;
    tl.start = uni(tp[4 * t]);
    tl.end = uni(tp[4 * t + 1]);
    tl.row = uni(tp[4 * t + 2]);
    tl.c0c1 = uni(tp[4 * t + 3]);
    if (tl.end <= tl.start) {  // empty slots are not tiles
        if (lane == 0) key[t] = kNoTile;
        return;
    }
    const TileStencil ts = tile_stencil<SPH>(P, tl);
    uint64_t nb = 0;
    for (int e = lane; e < ts.nrows; e += 64) {
        const RowSpans r = row_spans<SPH>(P, ts, e);
        nb += (r.a1 > r.a0 ? r.a1 - r.a0 : 0u) + (r.b1 > r.b0 ? r.b1 - r.b0 : 0u);
        nb += (r.m1 > tl.start ? r.m1 - tl.start : 0u) + (r.h1 - r.h0);
    }
    for (int off = 32; off > 0; off >>= 1) nb += __shfl_xor(nb, off);
    if (lane == 0) {
        // bucket on a log scale, 8 per octave, largest cost first (bucket 0);
        // log2(c) is in [11, 64)
        const uint64_t c = (uint64_t)(tl.end - tl.start) * nb + 32ull * (uint32_t)ts.nrows + 2048ull;
        const float lc = (__builtin_amdgcn_logf((float)c) - 11.0f) * 8.0f;
        key[t] = kCostBuckets - 1u - (uint32_t)fminf(fmaxf(lc, 0.0f), (float)(kCostBuckets - 1));
    }
}

// Rank of each tile within its bucket: LDS atomics inside the block, then one
// global atomic per (block, bucket) reserves the block's range. (A thread past
// the end or on an empty slot joins the barriers and counts nothing.)
__global__ __launch_bounds__(256) void k_tile_rank(const uint32_t* __restrict__ key, uint32_t ntiles,
                                                   uint32_t* __restrict__ rank,
                                                   uint32_t* __restrict__ hist) {
    const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t b = t < ntiles ? key[t] : kNoTile;
    const bool live = b != kNoTile;
    __shared__ uint32_t lh[kCostBuckets], lbase[kCostBuckets];
    for (uint32_t i = threadIdx.x; i < kCostBuckets; i += blockDim.x) lh[i] = 0u;
    __syncthreads();
    const uint32_t lr = live ? atomicAdd(&lh[b], 1u) : 0u;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < kCostBuckets; i += blockDim.x)
        if (lh[i]) lbase[i] = atomicAdd(&hist[i], lh[i]);
    __syncthreads();
    if (live) rank[t] = lbase[b] + lr;
}

// Parts per home tile (log2), from the tiles' costs (one bucket per thread: v
// tiles of cost c, upto of them up to this bucket; all threads of one block).
// pc.slots waves take the tasks longest first. A task of a full chip takes its
// pairs and its set-up, at least the set-up's waits beside which pairs of other
// waves are issued (own); one that starts when the tasks before it are shared
// out ends at (theirs and its own) / slots + own. The tasks that are their
// waves' first run on while others have ended, faster; when all of them are, or
// nearly all, some CUs have more of them than others (a chip half full takes
// twice the time of an even share; a radial count of 5126 tiles on 5120 waves
// took 1.78 ms uncut and 1.58 in eight parts). The count ends at the latest of these, and the rule takes
// the cut that ends first.
// Costs are the device's because a host estimate sees the bounding box only:
// with one, a light-cone FP64 count of 2e5 points, mostly empty box, was left
// uncut and took 3.9 ms (1.9 in four parts), and an r-mu count of 3e5 with 15
// points a tile was cut into four parts and took 1.06 ms (0.50 uncut).
__device__ __forceinline__ uint32_t part_rule(uint32_t v, float c, uint32_t upto, uint32_t ntiles,
                                              const PartCost& pc) {
    constexpr int P = kMaxPartLog + 1, W = kCostBuckets / 64;
    __shared__ float wsum[W][P], wend[W][P];
    const int lane = (int)(threadIdx.x & 63u);
    const uint32_t wave = threadIdx.x >> 6;
    const float slots = (float)pc.slots, is = 1.0f / slots;
    float own[P], sum[P];
#pragma unroll
    for (int p = 0; p < P; p++) {
        const float n = (float)(1u << p);
        own[p] = fmaxf(c / n + pc.issue, 0.3f * (c / n) + pc.wait);
        sum[p] = (float)v * n * own[p];
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1)
#pragma unroll
        for (int p = 0; p < P; p++) {
            const float u = __shfl_up(sum[p], o);
            sum[p] += lane >= o ? u : 0.f;
        }
    if (lane == 63)
#pragma unroll
        for (int p = 0; p < P; p++) wsum[wave][p] = sum[p];
    __syncthreads();
    float end[P];
#pragma unroll
    for (int p = 0; p < P; p++) {
        const float n = (float)(1u << p);
        float all = 0.f;
        for (uint32_t w = 0; w < W; w++) {
            sum[p] += w < wave ? wsum[w][p] : 0.f;
            all += wsum[w][p];
        }
        end[p] = v == 0u ? 0.f : (float)upto * n > slots ? own[p] + sum[p] * is : pc.first * (c / n) + pc.wait;
        end[p] = fmaxf(end[p], all * (0.6f * is + 0.75f / ((float)ntiles * n)));
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
        for (int p = 0; p < P; p++) end[p] = fmaxf(end[p], __shfl_xor(end[p], o));
    if (lane == 0)
#pragma unroll
        for (int p = 0; p < P; p++) wend[wave][p] = end[p];
    __syncthreads();
    uint32_t best = 0;
    float least = 0.f;
    for (int p = 0; p < P; p++) {
        // (past some dozens of tasks per wave no cut is worth its parts)
        if (p > 0 && (float)ntiles * (float)(1u << p) > 64.0f * slots) break;
        float e = 0.f;
        for (uint32_t w = 0; w < W; w++) e = fmaxf(e, wend[w][p]);
        if (p == 0 || e < 0.98f * least) {
            best = (uint32_t)p;
            least = e;
        }
    }
    return best;
}

// The offsets of the buckets in the ordered list (a block of one thread per
// bucket, which holds v tiles); total, when set, receives the number of tiles
// and the log2 of their parts.
__device__ __forceinline__ void bucket_offsets(uint32_t v, uint32_t* off, uint32_t* total, const PartCost& pc) {
    static_assert(kCostBuckets == 256, "one bucket per thread");
    __shared__ uint32_t wsum[kCostBuckets / 64];
    const int lane = (int)(threadIdx.x & 63u);
    const uint32_t wave = threadIdx.x >> 6;
    const uint32_t incl = wave_incl_scan(v, lane);
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    uint32_t base = 0, n = 0;
    for (uint32_t w = 0; w < kCostBuckets / 64; w++) {
        base += w < wave ? wsum[w] : 0u;
        n += wsum[w];
    }
    off[threadIdx.x] = base + incl - v;
    if (total != nullptr) {
        const float c = __builtin_amdgcn_exp2f(11.0f + ((float)(kCostBuckets - 1 - threadIdx.x) + 0.5f) * 0.125f);
        const uint32_t p = part_rule(v, c, base + incl, n, pc);
        if (threadIdx.x == 0) {
            total[0] = n;
            total[1] = p;
        }
    }
}

// Scatter the tiles into bucket order: every block scans the bucket counts in
// LDS (kCostBuckets of them), then each tile goes to its bucket's offset plus
// its rank within the bucket. total: the number of tiles and the log2 of their
// parts, by one more block beside the others (by block 0, before its tiles, the
// kernel took 4.6 us, 4.3 so).
__global__ __launch_bounds__(256) void k_tile_scatter(const Tile* __restrict__ tiles, uint32_t ntiles,
                                                      const uint32_t* __restrict__ key,
                                                      const uint32_t* __restrict__ rank,
                                                      const uint32_t* __restrict__ hist,
                                                      Tile* __restrict__ out,
                                                      uint32_t* __restrict__ total, PartCost pc) {
    __shared__ uint32_t off[kCostBuckets];
    bucket_offsets(hist[threadIdx.x], off, blockIdx.x == gridDim.x - 1u ? total : nullptr, pc);
    __syncthreads();
    const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= ntiles) return;
    const uint32_t b = key[t];
    if (b == kNoTile) return;  // an empty slot
    out[off[b] + rank[t]] = tiles[t];
}

}  // namespace

// Reorder tiles longest first (estimated cost, descending): the persistent
// waves take the heavy tiles early and the light ones fill the tail.
cute_status order_tiles_to(const CountArgs& a, const Tile* in, uint32_t ntiles, const PartCost& pc, uint32_t* key,
                           uint32_t* rank, uint32_t* hist, Tile* out, uint32_t* total, hipStream_t s) {
    static_assert(kCostBuckets == kTileBuckets, "one count per bucket");
    const unsigned nb = (ntiles + 255u) / 256u;
    auto cost = a.geom == CUTE_GEOM_SPHERE ? k_tile_cost<true> : k_tile_cost<false>;
    hipLaunchKernelGGL(cost, dim3((ntiles + 3u) / 4u), dim3(256), 0, s, a, in, ntiles, key);
    CUTE_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_tile_rank, dim3(nb), dim3(256), 0, s, key, ntiles, rank, hist);
    CUTE_HIP(hipGetLastError());
    hipLaunchKernelGGL(k_tile_scatter, dim3(nb + 1u), dim3(256), 0, s, in, ntiles, key, rank, hist, out, total, pc);
    CUTE_HIP(hipGetLastError());
    return CUTE_OK;
}

cute_status order_tiles(const CountArgs& a, Tile** tiles, uint32_t ntiles, const PartCost& pc, uint32_t* total,
                        hipStream_t s) {
    if (ntiles == 0) return CUTE_OK;
    TempList tmp(s);
    uint32_t* w = nullptr;   // keys | ranks | bucket counts
    Tile* t1 = nullptr;
    cute_status st;
    if ((st = tmp.alloc(&w, 2 * (size_t)ntiles + kTileBuckets)) != CUTE_OK) return st;
    uint32_t* hist = w + 2 * (size_t)ntiles;
    if ((st = zero_u32(hist, kTileBuckets, s)) != CUTE_OK) return st;
    if ((st = dalloc(&t1, ntiles, s)) != CUTE_OK) return st;
    if ((st = order_tiles_to(a, *tiles, ntiles, pc, w, w + ntiles, hist, t1, total, s)) != CUTE_OK) {
        dfree(t1, s);
        return st;
    }
    dfree(*tiles, s);
    *tiles = t1;
    return CUTE_OK;
}

cute_status build_tiles(const GridHost& g, int max_w, hipStream_t s, Tile** tiles,
                        uint32_t* ntiles) {
    *tiles = nullptr;
    *ntiles = 0;
    const int nrows = g.ny * g.nz;
    TempList tmp(s);
    uint32_t* cnt = nullptr;
    cute_status st = tmp.alloc(&cnt, (size_t)nrows + 1);
    if (st != CUTE_OK) return st;
    const unsigned nb = (unsigned)((nrows + 255) / 256);
    hipLaunchKernelGGL(k_tiles_count, dim3(nb), dim3(256), 0, s, g.cstart, g.nx, nrows, max_w,
                       (uint32_t)g.tile_max, cnt);
    CUTE_HIP(hipGetLastError());
    if ((st = exclusive_scan(cnt, cnt, (size_t)nrows + 1, s)) != CUTE_OK) return st;
    uint32_t total = 0;
    CUTE_HIP(hipMemcpyAsync(&total, cnt + nrows, sizeof(uint32_t), hipMemcpyDeviceToHost, s));
    CUTE_HIP(hipStreamSynchronize(s));
    Tile* t = nullptr;
    if ((st = dalloc(&t, total, s)) != CUTE_OK) return st;
    if (total > 0) {
        hipLaunchKernelGGL(k_tiles_write, dim3(nb), dim3(256), 0, s, g.cstart, g.nx, nrows,
                           max_w, (uint32_t)g.tile_max, cnt, t, (uint32_t*)nullptr);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) {
            dfree(t, s);
            return hip_status(e, "tiles launch");
        }
    }
    *tiles = t;
    *ntiles = total;
    return CUTE_OK;
}

cute_status region_tiles(const GridHost& g, int max_w, const uint32_t* rc, uint32_t K, uint32_t* off,
                         uint32_t* fill, Tile* out, hipStream_t s) {
    const int nrows = g.ny * g.nz;
    const unsigned nb = (unsigned)((nrows + 3) / 4);  // one wave per row
    const int w = max_w < 1 ? 1 : max_w;
    cute_status st = zero_u32(out ? fill : off, out ? (size_t)K : (size_t)K + 1, s);
    if (st != CUTE_OK) return st;
    if (out)
        hipLaunchKernelGGL(k_region_tiles<true>, dim3(nb), dim3(256), 0, s, g.cstart, g.nx, nrows, w,
                           (uint32_t)g.tile_max, rc, fill, off, out);
    else
        hipLaunchKernelGGL(k_region_tiles<false>, dim3(nb), dim3(256), 0, s, g.cstart, g.nx, nrows, w,
                           (uint32_t)g.tile_max, rc, off, nullptr, nullptr);
    CUTE_HIP(hipGetLastError());
    return out ? CUTE_OK : exclusive_scan(off, off, (size_t)K + 1, s);
}

// In a row, a tile is opened by the row's first point, after a tile of tmax
// points (at most floor(points / tmax) times) or when the next point lies
// max_w cells or more past the open tile's first cell (the first cell then
// advances by at least max_w: at most floor((nx - 1) / max_w) times).
uint64_t tile_count_bound(const GridHost& g, int max_w) {
    const uint64_t rows = (uint64_t)g.ny * (uint64_t)g.nz;
    const uint64_t w = (uint64_t)(max_w < 1 ? 1 : max_w);
    return (uint64_t)g.n / (uint64_t)g.tile_max + rows * ((uint64_t)(g.nx - 1) / w + 1u);
}

cute_status tiles_to_slots(const GridHost& g, int max_w, uint32_t bound, Tile* t, uint32_t* overflow,
                           uint32_t* total, hipStream_t s) {
    const int nrows = g.ny * g.nz;
    const unsigned nb = (unsigned)((nrows + 3) / 4);  // one wave per row
    hipLaunchKernelGGL(k_tiles_sparse, dim3(nb), dim3(256), 0, s, g.cstart, g.nx, nrows,
                       max_w < 1 ? 1 : max_w, (uint32_t)g.tile_max, t, bound, overflow, total);
    CUTE_HIP(hipGetLastError());
    return CUTE_OK;
}

}  // namespace cute
