// Batched pair counts: many (grid, grid, mask) items that share one binning in
// one persistent launch.
//
// A workgroup works on one item at a time, so its shared LDS histogram always
// holds counts of a single item: it starts with the item that the host's
// cost estimates give it, its waves pop tasks (parts of home tiles) from that
// item's own counter until none is left, and only then it sums its histogram
// into the item's global counts and moves to the item with the most tasks
// left. The waves meet at a barrier once per item: with chunks of four tiles
// handed to whole workgroups they met after every tile, and waited for the
// slowest of four (region pass of 100 regions and 2.5e5 points: 4.4 ms, 3.6
// with the items' own counters). Point masks (bits in sorted order) leave excluded home
// points and neighbour lanes idle.
#include <type_traits>

#include "count_device.h"

namespace cute {

namespace {

// Sum the workgroup's histogram copies into counts (one atomic per non-empty
// bin) and clear them (counters of 4 bytes when H32, else 8; with hi set, the
// high halves go there).
template <bool H32>
__device__ void flush_hist(unsigned char* hist0, int nbins, int copies, unsigned long long* counts,
                           unsigned long long* hi) {
    typedef typename std::conditional<H32, uint32_t, unsigned long long>::type word;
    for (int b = threadIdx.x; b < nbins; b += blockDim.x) {
        uint64_t s = 0, t = 0;
        word* hh = reinterpret_cast<word*>(hist0) + (size_t)b * copies;
        for (int c = 0; c < copies; c++) {
            const uint64_t w = hh[c];
            s += H32 || hi == nullptr ? w : (uint64_t)(uint32_t)w;
            if (!H32 && hi != nullptr) t += w >> 32;
            hh[c] = 0;
        }
        if (s) atomicAdd(&counts[b], (unsigned long long)s);
        if (t) atomicAdd(&hi[b], (unsigned long long)t);
    }
}

// The entry of the list to go on with (one wave): of the first 64 entries
// after pos, cyclically, with any task left, the one with the most; kNoBin
// when every item's tasks are taken.
__device__ __forceinline__ uint32_t next_item(const BatchArgs& BA, uint32_t pos, int lane) {
    const uint32_t n = BA.nlist;
    if (uni((uint32_t)__hip_atomic_load(BA.done, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) >= n) return kNoBin;
    for (uint32_t o = 0; o < n; o += 64u) {
        uint32_t e = 0, left = 0;
        if (o + (uint32_t)lane < n) {
            e = (uint32_t)(((uint64_t)pos + 1u + o + (uint32_t)lane) % n);
            const uint32_t item = BA.list[e], all = BA.ntiles[2u * item] << BA.ntiles[2u * item + 1u];
            const uint32_t head = (uint32_t)__hip_atomic_load(BA.heads + item, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            left = head < all ? all - head : 0u;
        }
        uint32_t m = left;
        for (int k = 32; k > 0; k >>= 1) {
            const uint32_t u = (uint32_t)__shfl_xor((int)m, k);
            m = u > m ? u : m;
        }
        if (m != 0u) return lane_u32(e, __builtin_ctzll(__builtin_amdgcn_ballot_w64(left == m)));
    }
    return kNoBin;
}

template <int MODE, int PREC, int EST>
__global__ __launch_bounds__(256, (kWgPerCu<MODE, PREC>)) void k_count_batch(BatchArgs BA) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int nwaves = blockDim.x >> 6;
    const int n1 = BA.n1;
    const int n2p = BA.n2 > 0 ? BA.n2 : 0;
    constexpr bool H32 = kH32<MODE>;
    const WgLds L = wg_lds<H32, kMfma<MODE, PREC, EST>, kAlpha<MODE>>(smem, nwaves, n1, BA.n2, BA.hist_words);
    double *T1 = L.T1, *T2 = L.T2;
    float2 *B1 = L.B1, *B2 = L.B2;
    unsigned char* hist0 = L.hist;
    uint32_t* ctl = L.ctl;        // [0] the next entry of the list
    uint32_t* budget = H32 ? ctl + 4 : ctl + 1;   // 32-bit counters and pairs of them
    for (int i = threadIdx.x; i <= n1; i += blockDim.x) T1[i] = BA.T1[i];
    for (int i = threadIdx.x; i <= n2p; i += blockDim.x) T2[i] = n2p ? BA.T2[i] : 0.0;
    if (PREC != P_FP64) {
        // (sigma-pi from the matrix cores: one entry past the last bin)
        constexpr int more = kMfma<MODE, PREC, EST> && MODE == M_SIGMAPI ? 1 : 0;
        for (int i = threadIdx.x; i < n1 + more; i += blockDim.x) B1[i] = BA.band1[i];
        for (int i = threadIdx.x; i < n2p + more; i += blockDim.x) B2[i] = BA.band2[i];
    }
    for (size_t i = threadIdx.x; i < L.hbytes / 4; i += blockDim.x) reinterpret_cast<uint32_t*>(hist0)[i] = 0u;
    for (int i = threadIdx.x; i < 2 * nwaves; i += blockDim.x) L.rstat[i] = 0ull;
    if (threadIdx.x == 0) *budget = 0u;

    WaveState W = wave_state(L, wave);
    W.budget = budget;
    SpanBuf S = span_buf(L, wave);

    __syncthreads();
    const cu32p list = (cu32p)(const void*)BA.list, ntl = (cu32p)(const void*)BA.ntiles;
    uint32_t pos = ((cu32p)(const void*)BA.first)[blockIdx.x];
    while (pos != kNoBin) {
        const uint32_t item = uni(list[pos]);
        const CountArgs& P = *(const CountArgs*)(cargp)(uintptr_t)(BA.items + item);
        const uint32_t plog = uni(ntl[2u * item + 1u]), ntasks = uni(ntl[2u * item]) << plog;
        uint32_t* head = reinterpret_cast<uint32_t*>(BA.heads + item);
        bool any = false;
        for (;;) {
            uint32_t t = 0;
            if (lane == 0) t = atomicAdd(head, 1u);
            t = uni(t);
            if (t >= ntasks) {
                // the one pop that finds the item's end
                if (t == ntasks && lane == 0) atomicAdd(BA.done, 1ull);
                break;
            }
            any = true;
            const cu32p tp = (cu32p)(const void*)P.tiles + 4 * (size_t)(t >> plog);
            Tile tl;
            tl.start = uni(tp[0]);
            tl.end = uni(tp[1]);
            tl.row = uni(tp[2]);
            tl.c0c1 = uni(tp[3]);
            do_tile<MODE, PREC, EST, true, false>(P, W, S, B1, B2, T1, T2, lane, tl,
                                                  t & ((1u << plog) - 1u), plog);
        }
        if (any) {
            // the re-test queue refers to this item's points: empty it now
            if constexpr (PREC == P_FP32E)
                W.tail = drain_queue<MODE, EST>(P.self, W.hist, W.qi, W.qj, W.qc, W.rstat, B1, B2, T1, T2,
                                                lane, W.tail, true);
            if (lane == 0) {
                atomicAdd(&P.stats[0], (unsigned long long)W.evals);
                atomicAdd(&P.stats[1], W.rstat[0]);
                atomicAdd(&P.stats[2], W.rstat[1]);
                atomicAdd(&P.stats[3], (unsigned long long)W.tiles);
                W.rstat[0] = 0ull;
                W.rstat[1] = 0ull;
            }
            W.evals = W.tiles = 0;
            W.pend = 0;
        }
        // every wave is done with the item
        if (__syncthreads_or(any ? 1 : 0)) {
            flush_hist<H32>(hist0, BA.nbins, BA.copies, P.counts, P.counts_hi);
            if (threadIdx.x == 0) *budget = 0u;
        }
        if (wave == 0) {
            const uint32_t nx = next_item(BA, pos, lane);
            if (lane == 0) ctl[0] = nx;
        }
        __syncthreads();
        pos = uni(ctl[0]);
    }
}

// Sorted-order exclusion bits of a mask given in the caller's input order:
// bit i of word i / 32 is set when mask[idx of sorted point i] != 0.
__global__ __launch_bounds__(256) void k_mask_bits(const uint8_t* __restrict__ mask,
                                                   const P64* __restrict__ p64, uint32_t n,
                                                   uint32_t* __restrict__ bits) {
    const uint32_t w = blockIdx.x * blockDim.x + threadIdx.x;
    if ((uint64_t)w * 32u >= n) return;
    uint32_t b = 0;
    for (uint32_t k = 0; k < 32u; k++) {
        const uint32_t i = w * 32u + k;
        if (i < n && mask[p64[i].idx] != 0) b |= 1u << k;
    }
    bits[w] = b;
}

// Zero n 64-bit words (a kernel, so that captured graphs hold no memset).
__global__ __launch_bounds__(256) void k_zero_u64(unsigned long long* __restrict__ p, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0ull;
}

__global__ __launch_bounds__(256) void k_zero_u32(uint32_t* __restrict__ p, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n;
         i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

template <int MODE, int PREC, int EST>
cute_status prep_one(size_t lds, int* per_cu) {
    auto kern = k_count_batch<MODE, PREC, EST>;
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void*)kern,
                                           hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return hip_status(e, "hipFuncSetAttribute");
    }
    CUTE_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, kern, 64 * kWgWaves, lds));
    if (*per_cu < 1) *per_cu = 1;
    return CUTE_OK;
}

template <int MODE, int PREC, int EST>
cute_status launch_b(const BatchArgs& ba, int grid, size_t lds, hipStream_t s) {
    hipLaunchKernelGGL((k_count_batch<MODE, PREC, EST>), dim3(grid), dim3(64 * kWgWaves), lds, s, ba);
    CUTE_HIP(hipGetLastError());
    return CUTE_OK;
}

// Dispatch on (mode, prec, est) to F<MODE, PREC, EST>(args...).
#define CUTE_DISPATCH(FN, mode, prec, est, ...)                                              \
    do {                                                                                      \
        const int m_ = (mode), p_ = (prec), e_ = (est) & E_LOG;                               \
        if (p_ == P_FP32E && ((est) & (E_DIF | E_MUF)) != 0) {                                \
            switch (m_ * 8 + (est)) {                                                         \
                case 4: return FN<0, 1, 4>(__VA_ARGS__);                                      \
                case 5: return FN<0, 1, 5>(__VA_ARGS__);                                      \
                case 14: return FN<1, 1, 6>(__VA_ARGS__);                                     \
                case 15: return FN<1, 1, 7>(__VA_ARGS__);                                     \
                case 12: return FN<1, 1, 4>(__VA_ARGS__);                                     \
                case 13: return FN<1, 1, 5>(__VA_ARGS__);                                     \
                case 10: return FN<1, 1, 2>(__VA_ARGS__);                                     \
                case 11: return FN<1, 1, 3>(__VA_ARGS__);                                     \
                case 20: return FN<2, 1, 4>(__VA_ARGS__);                                     \
                case 21: return FN<2, 1, 5>(__VA_ARGS__);                                     \
                case 18: return FN<2, 1, 2>(__VA_ARGS__);                                     \
                case 19: return FN<2, 1, 3>(__VA_ARGS__);                                     \
                case 28: return FN<3, 1, 4>(__VA_ARGS__);                                     \
                case 36: return FN<4, 1, 4>(__VA_ARGS__);                                     \
                case 37: return FN<4, 1, 5>(__VA_ARGS__);                                     \
                default: return fail(CUTE_E_INTERNAL, "unknown kernel variant");              \
            }                                                                                 \
        }                                                                                     \
        switch (m_ * 6 + p_ * 2 + e_) {                                                       \
            case 0: return FN<0, 0, 0>(__VA_ARGS__);                                          \
            case 1: return FN<0, 0, 1>(__VA_ARGS__);                                          \
            case 2: return FN<0, 1, 0>(__VA_ARGS__);                                          \
            case 3: return FN<0, 1, 1>(__VA_ARGS__);                                          \
            case 4: return FN<0, 2, 0>(__VA_ARGS__);                                          \
            case 5: return FN<0, 2, 1>(__VA_ARGS__);                                          \
            case 6: return FN<1, 0, 0>(__VA_ARGS__);                                          \
            case 7: return FN<1, 0, 1>(__VA_ARGS__);                                          \
            case 10: return FN<1, 2, 0>(__VA_ARGS__);                                         \
            case 11: return FN<1, 2, 1>(__VA_ARGS__);                                         \
            case 12: return FN<2, 0, 0>(__VA_ARGS__);                                         \
            case 13: return FN<2, 0, 1>(__VA_ARGS__);                                         \
            case 16: return FN<2, 2, 0>(__VA_ARGS__);                                         \
            case 17: return FN<2, 2, 1>(__VA_ARGS__);                                         \
            case 18: return FN<3, 0, 0>(__VA_ARGS__);                                         \
            case 20: return FN<3, 1, 0>(__VA_ARGS__);                                         \
            case 22: return FN<3, 2, 0>(__VA_ARGS__);                                         \
            case 24: return FN<4, 0, 0>(__VA_ARGS__);                                         \
            case 25: return FN<4, 0, 1>(__VA_ARGS__);                                         \
            case 26: return FN<4, 1, 0>(__VA_ARGS__);                                         \
            case 27: return FN<4, 1, 1>(__VA_ARGS__);                                         \
            case 28: return FN<4, 2, 0>(__VA_ARGS__);                                         \
            case 29: return FN<4, 2, 1>(__VA_ARGS__);                                         \
            default: return fail(CUTE_E_INTERNAL, "unknown kernel variant");                  \
        }                                                                                     \
    } while (0)

}  // namespace

cute_status batch_prepare(int mode, int prec, int est, size_t lds, int* per_cu) {
    CUTE_DISPATCH(prep_one, mode, prec, est, lds, per_cu);
}

cute_status batch_launch(const BatchArgs& ba, int mode, int prec, int est, int grid, size_t lds,
                         hipStream_t s) {
    CUTE_DISPATCH(launch_b, mode, prec, est, ba, grid, lds, s);
}

cute_status mask_bits(const uint8_t* mask, const GridHost& g, uint32_t* bits, hipStream_t s) {
    const uint32_t words = (uint32_t)((g.n + 31) / 32);
    if (words == 0) return CUTE_OK;
    hipLaunchKernelGGL(k_mask_bits, dim3((words + 255) / 256), dim3(256), 0, s, mask, g.p64,
                       (uint32_t)g.n, bits);
    CUTE_HIP(hipGetLastError());
    return CUTE_OK;
}

cute_status zero_u64(unsigned long long* p, size_t n, hipStream_t s) {
    if (n == 0) return CUTE_OK;
    size_t blocks = (n + 255) / 256;
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(k_zero_u64, dim3((unsigned)blocks), dim3(256), 0, s, p, n);
    CUTE_HIP(hipGetLastError());
    return CUTE_OK;
}

cute_status zero_u32(uint32_t* p, size_t n, hipStream_t s) {
    if (n == 0) return CUTE_OK;
    size_t blocks = (n + 255) / 256;
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(k_zero_u32, dim3((unsigned)blocks), dim3(256), 0, s, p, n);
    CUTE_HIP(hipGetLastError());
    return CUTE_OK;
}

}  // namespace cute
