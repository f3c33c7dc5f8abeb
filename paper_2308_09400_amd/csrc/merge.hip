// Merging of duplicate constraints after staging.  On aligned grids many
// candidate tuples reduce to the same point-edge or point-point constraint
// (a point over a shared edge or vertex is found through every triangle and
// edge pair around it).  The energy of Eq. 3 sums each candidate with its
// own constrained distance, so identical reduced constraints can be
// evaluated once and weighted by their count: that is exact.
//
// Duplicates are found with an open-addressing hash table on a 64-bit
// fingerprint of the canonical key (PP: the unordered vertex pair; PE: the
// point and the unordered edge).  The representative of a key is the
// smallest staged index carrying it (atomicMin), and a pair merges into it
// only if its full key equals the representative's, so a fingerprint
// collision can only leave duplicates unmerged, never merge different
// constraints.  Counts are integer atomics and the compaction keeps the
// staged order, so the result is deterministic.
//
// One lane per group of equal keys in a wavefront goes to the table.  The
// insert keeps the slot it found for every pair and counts the group there,
// so the second pass only reads: the slot, and the representative's key.
//
// Layout: one 8-byte word per slot holding a 36-bit fingerprint above the
// 28-bit representative (staged indices are below 2^28), so a slot is
// claimed and its representative lowered with 64-bit atomics on one word
// (the minimum of two words with the same fingerprint is the one with the
// smaller representative).  A key's home slot is proportional to its first
// vertex plus a 16-slot offset from the fingerprint: staged pairs come in
// vertex-major order within each sub-type, so neighbouring lanes probe
// neighbouring lines.
#include "internal.hpp"

namespace gipc {
namespace {

// splitmix64 finalizer (Steele, Lea, Flood, "Fast splittable pseudorandom
// number generators", 2014)
__device__ __forceinline__ uint64_t mix64(uint64_t z) {
    z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
    z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
    return z ^ (z >> 31);
}

struct Key {
    int a, b, c;
};

__device__ __forceinline__ Key canon(bool pp, int4 v) {
    if (pp) return Key{min(v.x, v.y), max(v.x, v.y), -1};
    return Key{v.x, min(v.y, v.z), max(v.y, v.z)};
}

constexpr int kRepBits = 28;
constexpr unsigned long long kRepMask = (1ull << kRepBits) - 1ull;

// 36-bit fingerprint in the high bits of a slot word, never 0 (0 = empty)
__device__ __forceinline__ unsigned long long fingerprint(const Key& k) {
    uint64_t x = ((uint64_t)(uint32_t)k.a << 32) | (uint32_t)k.b;
    uint64_t f = mix64(x ^ mix64((uint64_t)(uint32_t)k.c + 0x9e3779b97f4a7c15ull)) & ~kRepMask;
    return f ? f : (1ull << kRepBits);
}

__device__ __forceinline__ uint64_t home(const Key& k, unsigned long long f, double scale, uint64_t mask) {
    return ((uint64_t)((double)(uint32_t)k.a * scale) + ((f >> kRepBits) & 15ull)) & mask;
}

// Probes stop after kMaxProbe slots: a group whose key finds neither its
// slot nor an empty one that close to home stands for itself (exact, only
// slower).
constexpr int kMaxProbe = 4096;

// pairs [k0, k1) are PE then PP from pp0 on.  slot[k - k0] = the key's slot,
// or ~leader where the probe bound was reached (the group then stands for
// itself); own[slot] = the pairs of the group that claimed it, cnt[slot] those
// of the others, lone those of a group without a slot, at its leader.  An
// atomic costs some 16 cycles of an L2 channel, a load one: a slot is read
// first, and only claiming it, lowering its representative (rare: pairs come
// in order) and counting into another group's slot are atomics.
__global__ void __launch_bounds__(kBlock) k_merge_insert(const int4* __restrict__ st_vid, int64_t k0, int64_t k1,
                                                         int64_t pp0, unsigned long long* __restrict__ table,
                                                         int32_t* __restrict__ cnt, int32_t* __restrict__ own,
                                                         double scale, uint64_t mask, int32_t* __restrict__ slot,
                                                         int32_t* __restrict__ lone) {
    __shared__ uint32_t tab[kBlock / 64][kGroupSlots];
    const int64_t k = k0 + (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const bool in = k < k1;
    const bool pp = k >= pp0;
    const Key key = in ? canon(pp, st_vid[k]) : Key{-1, -1, -1};
    // the kinds cannot meet: a PP key has c = -1
    const int kk[3] = {key.a, key.b, key.c};
    const WaveGroup grp = wave_group<3>(kk, in, tab[threadIdx.x >> 6]);
    const int lane = threadIdx.x & 63;
    int32_t found = ~(int32_t)k;
    if (in && grp.leader == lane) {
        const unsigned long long f = fingerprint(key);
        const unsigned long long word = f | (unsigned long long)k;
        uint64_t h = home(key, f, scale, mask);
        for (int t = 0; t < kMaxProbe; ++t) {
            unsigned long long prev = __hip_atomic_load(&table[h], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (prev == 0ull) {
                prev = atomicCAS(&table[h], 0ull, word);
                if (prev == 0ull) {
                    own[h] = grp.count;
                    found = (int32_t)h;
                    break;
                }
            }
            if ((prev & ~kRepMask) == f) {
                if (word < prev) atomicMin(&table[h], word);
                atomicAdd(&cnt[h], grp.count);
                found = (int32_t)h;
                break;
            }
            h = (h + 1) & mask;
        }
        if (found < 0) lone[k - k0] = grp.count;
    }
    found = __shfl(found, grp.leader < 0 ? lane : grp.leader, 64);
    if (in) slot[k - k0] = found;
}

// Staged pairs outside [k0, k1) survive with multiplicity 1.  Inside it,
// state[k - k0] (over slot) = 0 for a pair that merges into its key's
// representative, its multiplicity for one that stands for itself, and ~slot
// for a representative, whose multiplicity is own + cnt of the slot.  A pair whose
// key is not the representative's (a fingerprint collision) takes itself out
// of that count.  Survivors are counted per workgroup of kBlock pairs.
__global__ void __launch_bounds__(kBlock) k_merge_resolve(const int4* __restrict__ st_vid, int64_t Ps, int64_t k0,
                                                          int64_t k1, int64_t pp0,
                                                          const unsigned long long* __restrict__ table,
                                                          int32_t* __restrict__ cnt, int32_t* __restrict__ state,
                                                          const int32_t* __restrict__ lone,
                                                          int32_t* __restrict__ bcnt) {
    __shared__ int32_t wcnt[kBlock / 64];
    const int64_t blk = xcd_block();  // neighbours look up the same slots: 255 -> 214 us
    const int64_t k = blk * kBlock + threadIdx.x;
    bool keep = k < Ps;
    if (k >= k0 && k < k1) {
        const int32_t s = state[k - k0];
        int32_t m = 0;
        if (s >= 0) {
            const int32_t r = (int32_t)(table[s] & kRepMask);
            if (r == (int32_t)k) {
                m = ~s;
            } else {
                const bool pp = k >= pp0, rpp = r >= pp0;
                const Key me = canon(pp, st_vid[k]), o = canon(rpp, st_vid[r]);
                if (!(rpp == pp && o.a == me.a && o.b == me.b && o.c == me.c)) {
                    atomicAdd(&cnt[s], -1);
                    m = 1;
                }
            }
        } else if (~s == (int32_t)k) {
            m = lone[k - k0];
        }
        state[k - k0] = m;
        keep = m != 0;
    }
    const unsigned long long b = __ballot(keep);
    if ((threadIdx.x & 63) == 0) wcnt[threadIdx.x >> 6] = __popcll(b);
    __syncthreads();
    if (threadIdx.x == 0) {
        int32_t c = 0;
        for (int w = 0; w < kBlock / 64; ++w) c += wcnt[w];
        bcnt[blk] = c;
    }
}

// the pairs the compaction keeps
__device__ __forceinline__ bool survives(int64_t k, int64_t Ps, int64_t k0, int64_t k1,
                                         const int32_t* __restrict__ state) {
    return k < Ps && (k < k0 || k >= k1 || state[k - k0] != 0);
}

// stable compaction: a survivor's position is its workgroup's offset plus
// the survivors before it in the workgroup
__global__ void __launch_bounds__(kBlock) k_merge_scatter(int64_t Ps, int64_t k0, int64_t k1,
                                                          const int32_t* __restrict__ state,
                                                          const int32_t* __restrict__ cnt_in,
                                                          const int32_t* __restrict__ own,
                                                          const int64_t* __restrict__ boff,
                                                          const int4* __restrict__ st_vid,
                                                          const int32_t* __restrict__ st_src,
                                                          int4* __restrict__ vid_out, int32_t* __restrict__ src_out,
                                                          int32_t* __restrict__ mult_out, TypeRanges tr,
                                                          int64_t* __restrict__ type_off) {
    __shared__ int32_t cnt[kBlock / 64];
    // the last nine workgroups leave the merged types' offsets: type t's is
    // the number of survivors before o
    const int64_t t = (int64_t)blockIdx.x - ((int64_t)gridDim.x - 9);
    const int64_t o = t >= 0 ? tr.off[t] : Ps;
    const int64_t b = t >= 0 ? o / kBlock : (int64_t)blockIdx.x;
    const int64_t k = b * kBlock + threadIdx.x;
    const int wid = threadIdx.x >> 6;
    const bool f = k < o && survives(k, Ps, k0, k1, state);
    const unsigned long long m = __ballot(f);
    if ((threadIdx.x & 63) == 0) cnt[wid] = __popcll(m);
    __syncthreads();
    int64_t n = boff[b];
    if (t >= 0) {
        for (int v = 0; v < kBlock / 64; ++v) n += cnt[v];
        if (threadIdx.x == 0) type_off[t] = n;
        return;
    }
    if (!f) return;
    for (int v = 0; v < wid; ++v) n += cnt[v];
    n += __popcll(m & __lanemask_lt());
    vid_out[n] = st_vid[k];
    src_out[n] = st_src[k];
    int32_t w = 1;
    if (k >= k0 && k < k1) {
        w = state[k - k0];
        if (w < 0) w = own[~w] + cnt_in[~w];
    }
    mult_out[n] = w;
}

unsigned grid(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

}  // namespace

hipError_t merge_duplicates(gipc_ctx* ctx, int32_t V, hipStream_t s, int64_t* new_off_dev) {
    const TypeRanges& tr = ctx->ranges;
    const int64_t Ps = tr.off[8], k0 = tr.off[FT_PE], pp0 = tr.off[FT_PP], k1 = tr.off[FT_PP + 1];
    const int64_t n = k1 - k0;
    uint64_t H = 1024;
    while (H < (uint64_t)n + (uint64_t)n / 4) H <<= 1;
    // home slots spread over the whole table: V is the vertex count of the pair set
    const double scale = V > 0 ? (double)H / (double)V : 1.0;
    hipError_t e;
#define TRY(x)                          \
    do {                                \
        if ((e = (x)) != hipSuccess) return e; \
    } while (0)
    TRY(ensure(ctx->mkeys, sizeof(unsigned long long) * H));
    TRY(ensure(ctx->mrep_of, sizeof(int32_t) * (size_t)(n > 0 ? n : 1)));
    TRY(ensure(ctx->mcount, sizeof(int32_t) * (size_t)(n > 0 ? n : 1)));
    const int64_t nbk = (Ps + kBlock - 1) / kBlock;  // compaction workgroups
    TRY(ensure(ctx->mbcount, sizeof(int32_t) * (size_t)(nbk > 0 ? nbk : 1)));
    TRY(ensure(ctx->mpos, sizeof(int64_t) * (size_t)(nbk + 1)));
    TRY(ensure(ctx->st_vid2, sizeof(int4) * (size_t)(Ps > 0 ? Ps : 1)));
    TRY(ensure(ctx->st_src2, sizeof(int32_t) * (size_t)(Ps > 0 ? Ps : 1)));
    TRY(ensure(ctx->mult, sizeof(int32_t) * (size_t)(Ps > 0 ? Ps : 1)));
    TRY(ensure(ctx->mslots, sizeof(int32_t) * 2 * H));
    int32_t *state = as<int32_t>(ctx->mrep_of), *count = as<int32_t>(ctx->mslots), *lone = as<int32_t>(ctx->mcount);
    int32_t* own = count + H;
    const unsigned long long* table = as<unsigned long long>(ctx->mkeys);
    if (n > 0) {
        ZeroList z;
        z.p[0] = as<int32_t>(ctx->mkeys), z.n[0] = 2 * (int64_t)H;
        z.p[1] = count, z.n[1] = (int64_t)H;
        TRY(zero_i32(z, s));
        k_merge_insert<<<grid(n), kBlock, 0, s>>>(as<int4>(ctx->st_vid), k0, k1, pp0,
                                                  as<unsigned long long>(ctx->mkeys), count, own, scale, H - 1,
                                                  state, lone);
        TRY(hipGetLastError());
    }
    if (Ps > 0) {
        k_merge_resolve<<<(unsigned)nbk, kBlock, 0, s>>>(as<int4>(ctx->st_vid), Ps, k0, k1, pp0, table, count, state,
                                                         lone, as<int32_t>(ctx->mbcount));
        TRY(hipGetLastError());
    }
    TRY((exclusive_scan<int32_t, int64_t>(as<int32_t>(ctx->mbcount), nbk, as<int64_t>(ctx->mpos), ctx, s)));
    if (Ps > 0) {
        k_merge_scatter<<<(unsigned)(nbk + 9), kBlock, 0, s>>>(
            Ps, k0, k1, state, count, own, as<int64_t>(ctx->mpos), as<int4>(ctx->st_vid), as<int32_t>(ctx->st_src),
            as<int4>(ctx->st_vid2), as<int32_t>(ctx->st_src2), as<int32_t>(ctx->mult), tr, new_off_dev);
        TRY(hipGetLastError());
    }
#undef TRY
    std::swap(ctx->st_vid, ctx->st_vid2);
    std::swap(ctx->st_src, ctx->st_src2);
    return hipSuccess;
}

}  // namespace gipc
