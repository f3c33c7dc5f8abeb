// Device-wide exclusive scan: block sums, scan of the block sums in one
// workgroup, block-local scans plus carry.  Up to kScanFold blocks every
// block of the last pass adds the sums before it by itself, which saves the
// launch in the middle (a build of two 128 x 128 sheets 295 against 319 us, of
// two 181 x 181 381 against 409).  Up to kScanOne elements, two rounds of its
// loop, one workgroup does everything in one launch: builds of two sheets of
// 4050 vertices in all 200 us against 213 with two launches, of 5000 212
// against 209 (with a line above them), of 16200 290 against 244.
// Integer arithmetic only, so the results are deterministic.
#include "internal.hpp"

namespace gipc {
namespace {

constexpr int kChunk = kBlock * kScanItems;  // elements per workgroup

template <typename T>
__device__ T block_exscan(T v, T* lds, T& total) {
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    T inc = v;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        T n = __shfl_up(inc, o, 64);
        if (lane >= o) inc += n;
    }
    if (lane == 63) lds[wid] = inc;
    __syncthreads();
    if (threadIdx.x == 0) {
        T s = 0;
        for (int w = 0; w < kBlock / 64; ++w) {
            T t = lds[w];
            lds[w] = s;
            s += t;
        }
        lds[kBlock / 64] = s;
    }
    __syncthreads();
    T ex = lds[wid] + inc - v;
    total = lds[kBlock / 64];
    __syncthreads();
    return ex;
}

template <typename TIn>
__global__ void __launch_bounds__(kBlock) k_scan_partial(const TIn* __restrict__ in, int64_t n,
                                                         int64_t* __restrict__ bsum) {
    __shared__ int64_t lds[kBlock / 64 + 1];
    int64_t base = (int64_t)blockIdx.x * kChunk + (int64_t)threadIdx.x * kScanItems;
    int64_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        int64_t i = base + k;
        if (i < n) s += (int64_t)in[i];
    }
    int64_t tot;
    block_exscan<int64_t>(s, lds, tot);
    if (threadIdx.x == 0) bsum[blockIdx.x] = tot;
}

// exclusive scan of bsum[0..nb) in place by one workgroup; out[n] = total
template <typename TOut>
__global__ void __launch_bounds__(kBlock) k_scan_top(int64_t* __restrict__ bsum, int64_t nb, TOut* __restrict__ out,
                                                     int64_t n, int64_t* __restrict__ total) {
    __shared__ int64_t lds[kBlock / 64 + 1];
    int64_t carry = 0;
    for (int64_t c0 = 0; c0 < nb; c0 += kChunk) {
        int64_t base = c0 + (int64_t)threadIdx.x * kScanItems;
        int64_t v[kScanItems];
        int64_t s = 0;
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            int64_t i = base + k;
            v[k] = i < nb ? bsum[i] : 0;
            s += v[k];
        }
        int64_t tot;
        int64_t ex = block_exscan<int64_t>(s, lds, tot) + carry;
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            int64_t i = base + k;
            if (i < nb) bsum[i] = ex;
            ex += v[k];
        }
        carry += tot;
    }
    if (threadIdx.x == 0) {
        out[n] = (TOut)carry;
        if (total) *total = carry;
    }
}

// FOLD: bsum holds the blocks' own sums and each block adds those before it
// (the last one also writes the total); otherwise bsum is already scanned
template <typename TIn, typename TOut, bool FOLD>
__global__ void __launch_bounds__(kBlock) k_scan_final(const TIn* __restrict__ in, int64_t n,
                                                       const int64_t* __restrict__ bsum, TOut* __restrict__ out,
                                                       int64_t* __restrict__ total) {
    __shared__ int64_t lds[kBlock / 64 + 1];
    int64_t base = (int64_t)blockIdx.x * kChunk + (int64_t)threadIdx.x * kScanItems;
    int64_t carry = 0;
    if (FOLD) {
        int64_t p = 0;
        for (int64_t b = threadIdx.x; b < (int64_t)blockIdx.x; b += kBlock) p += bsum[b];
        block_exscan<int64_t>(p, lds, carry);
    } else {
        carry = bsum[blockIdx.x];
    }
    int64_t v[kScanItems];
    int64_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        int64_t i = base + k;
        v[k] = i < n ? (int64_t)in[i] : 0;
        s += v[k];
    }
    int64_t tot;
    int64_t ex = block_exscan<int64_t>(s, lds, tot) + carry;
#pragma unroll
    for (int k = 0; k < kScanItems; ++k) {
        int64_t i = base + k;
        if (i < n) out[i] = (TOut)ex;
        ex += v[k];
    }
    if (FOLD && blockIdx.x == gridDim.x - 1 && threadIdx.x == 0) {
        out[n] = (TOut)(carry + tot);
        if (total) *total = carry + tot;
    }
}

// the whole scan in one workgroup of kBlock threads
template <typename TIn, typename TOut>
__global__ void __launch_bounds__(kBlock) k_scan_one(const TIn* __restrict__ in, int64_t n, TOut* __restrict__ out,
                                                     int64_t* __restrict__ total) {
    __shared__ int64_t lds[kBlock / 64 + 1];
    int64_t carry = 0;
    for (int64_t c0 = 0; c0 < n; c0 += kChunk) {
        const int64_t base = c0 + (int64_t)threadIdx.x * kScanItems;
        int64_t v[kScanItems];
        int64_t s = 0;
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            const int64_t i = base + k;
            v[k] = i < n ? (int64_t)in[i] : 0;
            s += v[k];
        }
        int64_t tot;
        int64_t ex = block_exscan<int64_t>(s, lds, tot) + carry;
#pragma unroll
        for (int k = 0; k < kScanItems; ++k) {
            const int64_t i = base + k;
            if (i < n) out[i] = (TOut)ex;
            ex += v[k];
        }
        carry += tot;
    }
    if (threadIdx.x == 0) {
        out[n] = (TOut)carry;
        if (total) *total = carry;
    }
}

constexpr int64_t kScanOne = 4096;
constexpr int64_t kScanFold = 1024;

}  // namespace

template <typename TIn, typename TOut>
hipError_t exclusive_scan(const TIn* in, int64_t n, TOut* out, gipc_ctx* ctx, hipStream_t s, int64_t* total_dev) {
    if (n <= kScanOne) {
        k_scan_one<TIn, TOut><<<1, kBlock, 0, s>>>(in, n, out, total_dev);
        return hipGetLastError();
    }
    const int64_t nb = (n + kChunk - 1) / kChunk;
    hipError_t e = ensure(ctx->scan_tmp, sizeof(int64_t) * nb);
    if (e != hipSuccess) return e;
    int64_t* bsum = as<int64_t>(ctx->scan_tmp);
    k_scan_partial<TIn><<<(unsigned)nb, kBlock, 0, s>>>(in, n, bsum);
    if (nb <= kScanFold) {
        k_scan_final<TIn, TOut, true><<<(unsigned)nb, kBlock, 0, s>>>(in, n, bsum, out, total_dev);
    } else {
        k_scan_top<TOut><<<1, kBlock, 0, s>>>(bsum, nb, out, n, total_dev);
        k_scan_final<TIn, TOut, false><<<(unsigned)nb, kBlock, 0, s>>>(in, n, bsum, out, total_dev);
    }
    return hipGetLastError();
}

template hipError_t exclusive_scan<int32_t, int64_t>(const int32_t*, int64_t, int64_t*, gipc_ctx*, hipStream_t,
                                                     int64_t*);
template hipError_t exclusive_scan<int32_t, int32_t>(const int32_t*, int64_t, int32_t*, gipc_ctx*, hipStream_t,
                                                     int64_t*);
template hipError_t exclusive_scan<int64_t, int64_t>(const int64_t*, int64_t, int64_t*, gipc_ctx*, hipStream_t,
                                                     int64_t*);

namespace {
constexpr int kZeroInts = 4 * kBlock;  // ints of a workgroup

// 16 bytes per lane where the array allows it: bound by its stores (a build of
// ten 256 x 256 sheets, most of it the merge table: 60 us in two launches; 110
// us in four with one int per lane)
__global__ void __launch_bounds__(kBlock) k_zero_i32(ZeroList z, int64_t* __restrict__ counters, int nslots,
                                                     uint64_t ones) {
    if (blockIdx.x == 0 && (int)threadIdx.x < nslots) counters[threadIdx.x] = (ones >> threadIdx.x) & 1u ? -1 : 0;
    int64_t b = blockIdx.x;
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        const int64_t nb = (z.n[a] + kZeroInts - 1) / kZeroInts;
        if (b >= 0 && b < nb) {
            const int64_t i = b * kZeroInts + 4 * threadIdx.x;
            if ((reinterpret_cast<uintptr_t>(z.p[a]) & 15u) == 0 && i + 4 <= z.n[a]) {
                *reinterpret_cast<int4*>(z.p[a] + i) = make_int4(0, 0, 0, 0);
            } else {
                for (int64_t j = i; j < i + 4 && j < z.n[a]; ++j) z.p[a][j] = 0;
            }
        }
        b -= nb;
    }
}
}  // namespace

hipError_t zero_i32(const ZeroList& z, hipStream_t s, int64_t* counters, int nslots, uint64_t ones) {
    int64_t nb = 0;
    for (int a = 0; a < 4; ++a) nb += (z.n[a] + kZeroInts - 1) / kZeroInts;
    if (nb == 0 && nslots == 0) return hipSuccess;
    k_zero_i32<<<(unsigned)(nb > 0 ? nb : 1), kBlock, 0, s>>>(z, counters, nslots, ones);
    return hipGetLastError();
}

}  // namespace gipc
