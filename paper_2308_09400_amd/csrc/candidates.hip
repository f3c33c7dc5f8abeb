// Contact candidates on the GPU: every point-triangle and edge-edge pair of
// different objects, sharing no vertex, whose axis-aligned boxes come within
// dhat (one box inflated by dhat, closed intervals) -- the pairs the sum of
// Eq. 3 ranges over, before the distance decides which are active.  A
// uniform grid stands in for the paper's LBVH (Sec. 7.2): along each axis
// the cell size is the largest primitive extent along that axis plus dhat,
// so every box spans at most two cells per axis, and thin stacks (sheets a
// fraction of dhat apart) are split along their normal; a pair is reported
// by the one cell holding the lower corner of its boxes' overlap, so each is
// found exactly once.
//
//  1. bounds: per-block minima / maxima of the positions and the largest
//     primitive extent, with a check of the vertex ids (the host finishes the
//     reduction and sizes the grid);
//  2. four cell tables numbered through: of the queries (points, then edges,
//     in the cells their box inflated by dhat covers, in any order) and of the
//     primitives (triangles, then edges): counts, one scan, one fill;
//  3. each primitive cell's list sorted by id, so the tables do not depend on
//     the order of the atomics;
//  4. one wave per cell pairing its queries with its primitives (points
//     against triangles, edges against edges of larger index): a counting
//     pass that also keeps the hit masks, a scan over the queries' visits
//     of cells, and an emitting pass that replays the masks.
// The output is deterministic: point-triangle candidates grouped by point in
// increasing order, then edge-edge candidates grouped by first edge, each
// group in cell order and primitive order within a cell.
#include "internal.hpp"

namespace gipc {
namespace {

struct Grid {
    double org[3];
    double h[3], inv[3];  // cell size and its reciprocal
    int32_t n[3];
};

struct Box {
    d3 lo, hi;
};

struct Prims {
    const int32_t *tris, *edges;
    int64_t F, E;
};

__host__ __device__ __forceinline__ int64_t blocks_of(int64_t n) { return (n + kBlock - 1) / kBlock; }

// one 64-byte record per primitive for the queries: its box, its vertex
// ids and its object, that of v[0]; v[2] also tells of vertices of different
// objects (triangles: ~v[2] in its place, edges: 1, otherwise 0)
struct __align__(64) PrimRec {
    double lo[3], hi[3];
    int32_t v[3];
    int32_t obj;
};

__device__ __forceinline__ Box prim_box(const double* __restrict__ X, const int32_t* v, int nper) {
    Box b{ld3(X, v[0]), ld3(X, v[0])};
    for (int k = 1; k < nper; ++k) {
        const d3 p = ld3(X, v[k]);
        b.lo = mk(fmin(b.lo.x, p.x), fmin(b.lo.y, p.y), fmin(b.lo.z, p.z));
        b.hi = mk(fmax(b.hi.x, p.x), fmax(b.hi.y, p.y), fmax(b.hi.z, p.z));
    }
    return b;
}

// floor((c - org) / h), clamped to the grid.  The product with the reciprocal
// is within 1.2e-7 of the quotient up to 2^28 cells, so it has the same floor
// unless it lies next to a whole number; only then is the division done.
__device__ __forceinline__ int cell_of(double c, const Grid& g, int d) {
    const double a = c - g.org[d];
    double f = a * g.inv[d], w = floor(f);
    if (!(f - w > 1e-6 && f - w < 1.0 - 1e-6)) w = floor(a / g.h[d]);
    const int i = (int)w;
    return i < 0 ? 0 : (i >= g.n[d] ? g.n[d] - 1 : i);
}

__device__ __forceinline__ double get(const d3& v, int d) { return d == 0 ? v.x : (d == 1 ? v.y : v.z); }

// box a inflated by dhat overlaps box b
__device__ __forceinline__ bool overlap(const Box& a, double dhat, const Box& b) {
    return !(a.lo.x - dhat > b.hi.x || b.lo.x > a.hi.x + dhat || a.lo.y - dhat > b.hi.y || b.lo.y > a.hi.y + dhat ||
             a.lo.z - dhat > b.hi.z || b.lo.z > a.hi.z + dhat);
}

// A wave's visits of cells flattened: each lane's cells lo..hi (x slowest,
// z fastest) are numbered after those of the lanes below it, and the wave
// takes them 64 at a time, so that lanes covering few cells do not idle
// while others walk up to 27.  f(cell, item, there) for every visit, by all
// lanes together; the owner of visit v is the last lane whose first number is
// at most v (a lane covering no cell shares its first number with the next
// lane and is never last).
template <typename C, typename F>
__device__ __forceinline__ void wave_visits(const int lo[3], const int hi[3], bool valid, int32_t item, C vcell, F f) {
    __shared__ int4 vbox[kBlock / 64][64];
    __shared__ int2 vnum[kBlock / 64][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int sy = hi[1] - lo[1] + 1, sz = hi[2] - lo[2] + 1;
    const int n = valid ? (hi[0] - lo[0] + 1) * sy * sz : 0;
    int inc = n;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int v = __shfl_up(inc, d, 64);
        if (lane >= d) inc += v;
    }
    const int total = __builtin_amdgcn_readlane(inc, 63);
    vbox[w][lane] = make_int4(lo[0], lo[1], lo[2], (sy << 8) | sz);
    vnum[w][lane] = make_int2(inc - n, item);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    for (int base = 0; base < total; base += 64) {
        const int v = base + lane;
        const bool in = v < total;
        int64_t cell = 0;
        int32_t who = 0;
        if (in) {
            int l = 0;
#pragma unroll
            for (int step = 32; step > 0; step >>= 1)
                if (vnum[w][l + step].x <= v) l += step;
            const int4 b = vbox[w][l];
            const int2 nm = vnum[w][l];
            const int bz = b.w & 255, byz = (b.w >> 8) * bz;
            const int j = v - nm.x;
            const int da = j / byz, rem = j - da * byz;
            const int dc = rem / bz, de = rem - dc * bz;
            cell = vcell(b.x + da, b.y + dc, b.z + de);
            who = nm.y;
        }
        f(cell, who, in);
    }
}

// per block: min x,y,z, max x,y,z of the positions, largest primitive extent
// along x, y, z, and the primitives with invalid vertex ids (out of range or
// repeated), which take no part in the extents: their number and the first of
// them, as integers.  One pass for both: the check by itself read the topology
// once more and its answer was waited for (a Newton step of two 16 x 16
// sheets 605 us, 640 with the pass of its own; ten 256 x 256 sheets'
// candidates 2930 and 2970).
__global__ void __launch_bounds__(kBlock) k_cand_bounds(const double* __restrict__ X, int32_t V, Prims pr,
                                                        CandBounds* __restrict__ part) {
    __shared__ double lds[kBlock / 64][9];
    __shared__ unsigned long long nbad, first;
    if (threadIdx.x == 0) {
        nbad = 0ull;
        first = ~0ull;
    }
    __syncthreads();
    double r[9] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY, 0.0, 0.0, 0.0};
    const int64_t stride = (int64_t)gridDim.x * kBlock, F = pr.F, E = pr.E;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < V; i += stride) {
        const d3 p = ld3(X, (int)i);
        r[0] = fmin(r[0], p.x); r[1] = fmin(r[1], p.y); r[2] = fmin(r[2], p.z);
        r[3] = fmax(r[3], p.x); r[4] = fmax(r[4], p.y); r[5] = fmax(r[5], p.z);
    }
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < F + E; i += stride) {
        const bool tri = i < F;
        const int32_t* v = tri ? pr.tris + 3 * i : pr.edges + 2 * (i - F);
        const int32_t a = v[0], b = v[1], c = tri ? v[2] : b;
        const bool ok = a >= 0 && a < V && b >= 0 && b < V && c >= 0 && c < V && a != b &&
                        (!tri || (c != a && c != b));
        if (!ok) {
            atomicAdd(&nbad, 1ull);
            atomicMin(&first, (unsigned long long)i);
            continue;
        }
        const Box x = tri ? prim_box(X, v, 3) : prim_box(X, v, 2);
        r[6] = fmax(r[6], x.hi.x - x.lo.x);
        r[7] = fmax(r[7], x.hi.y - x.lo.y);
        r[8] = fmax(r[8], x.hi.z - x.lo.z);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
#pragma unroll
        for (int q = 0; q < 3; ++q) r[q] = fmin(r[q], __shfl_xor(r[q], o, 64));
#pragma unroll
        for (int q = 3; q < 9; ++q) r[q] = fmax(r[q], __shfl_xor(r[q], o, 64));
    }
    if ((threadIdx.x & 63) == 0)
        for (int q = 0; q < 9; ++q) lds[threadIdx.x >> 6][q] = r[q];
    __syncthreads();
    if (threadIdx.x < 9) {
        const int q = threadIdx.x;
        double v = lds[0][q];
        for (int w = 1; w < kBlock / 64; ++w) v = q < 3 ? fmin(v, lds[w][q]) : fmax(v, lds[w][q]);
        part[blockIdx.x].r[q] = v;
    }
    if (threadIdx.x == 0) {
        part[blockIdx.x].nbad = (int64_t)nbad;
        part[blockIdx.x].first = (int64_t)first;
    }
}

// The four cell tables are counted and filled with one atomic per cell and
// wavefront's 64 visits: neighbouring primitives cover the same cells, and the
// passes are bound by their atomics (ten 256 x 256 sheets, 29 M visits: the
// four counts 495 -> 235 us and the four fills 625 -> 390 us against one
// atomic per visit).
__device__ __forceinline__ void count_visit(int64_t cell, bool there, int32_t* __restrict__ count, uint32_t* tab) {
    const int key[1] = {(int)cell};  // at most 2^28 cells
    const WaveGroup grp = wave_group<1>(key, there, tab);
    if (there && grp.leader == (int)(threadIdx.x & 63)) atomicAdd(&count[cell], grp.count);
}

__device__ __forceinline__ void fill_visit(int64_t cell, int32_t item, bool there, const int64_t* __restrict__ off,
                                           int32_t* __restrict__ fill, int32_t* __restrict__ ent, uint32_t* tab) {
    const int key[1] = {(int)cell};
    const WaveGroup grp = wave_group<1>(key, there, tab);
    int at = 0;
    if (there && grp.leader == (int)(threadIdx.x & 63)) at = atomicAdd(&fill[cell], grp.count);
    at = __shfl(at, there ? grp.leader : 0, 64);
    if (there) ent[off[cell] + at + grp.rank] = item;
}

// The queries' side, one record per query primitive: KIND 0 = points (their
// position, a zero-size box), 1 = edges (their 64-byte record).
template <int KIND>
__device__ __forceinline__ void query_of(int64_t q, const double* __restrict__ X, const int32_t* __restrict__ vobj,
                                         const PrimRec* __restrict__ qrec, Box& qb, int32_t& q0, int32_t& q1,
                                         int32_t& qo) {
    if (KIND == 0) {
        qb.lo = qb.hi = ld3(X, (int)q);
        q0 = q1 = (int32_t)q;
        qo = vobj[q];
    } else {
        const PrimRec r = qrec[q];
        qb.lo = mk(r.lo[0], r.lo[1], r.lo[2]);
        qb.hi = mk(r.hi[0], r.hi[1], r.hi[2]);
        q0 = r.v[0]; q1 = r.v[1]; qo = r.obj;
    }
}

// the cells covered by a query's box inflated by dhat
__device__ __forceinline__ void query_cells(const Box& qb, const Grid& g, double dhat, int lo[3], int hi[3]) {
    for (int d = 0; d < 3; ++d) {
        lo[d] = cell_of(get(qb.lo, d) - dhat, g, d);
        hi[d] = cell_of(get(qb.hi, d) + dhat, g, d);
    }
}

template <int NPER>
__device__ __forceinline__ void prim_record(const double* __restrict__ X, const int32_t* __restrict__ v,
                                            const int32_t* __restrict__ vobj, PrimRec* __restrict__ rec) {
    const Box b = prim_box(X, v, NPER);
    PrimRec r;
    r.lo[0] = b.lo.x; r.lo[1] = b.lo.y; r.lo[2] = b.lo.z;
    r.hi[0] = b.hi.x; r.hi[1] = b.hi.y; r.hi[2] = b.hi.z;
    const bool mixed = vobj[v[0]] != vobj[v[1]] || (NPER == 3 && vobj[v[0]] != vobj[v[NPER - 1]]);
    r.v[0] = v[0]; r.v[1] = v[1];
    r.v[2] = NPER == 3 ? (mixed ? ~v[2] : v[2]) : mixed;
    r.obj = vobj[v[0]];
    *rec = r;
}

// workgroups of the triangles first, then of the edges
__global__ void __launch_bounds__(kBlock) k_prim_records(const double* __restrict__ X, Prims pr,
                                                         const int32_t* __restrict__ vobj,
                                                         PrimRec* __restrict__ trec, PrimRec* __restrict__ erec) {
    const int64_t nt = blocks_of(pr.F);
    const bool tri = (int64_t)blockIdx.x < nt;
    const int64_t i = ((int64_t)blockIdx.x - (tri ? 0 : nt)) * kBlock + threadIdx.x;
    if (i >= (tri ? pr.F : pr.E)) return;
    if (tri) prim_record<3>(X, pr.tris + 3 * i, vobj, trec + i);
    else prim_record<2>(X, pr.edges + 2 * i, vobj, erec + i);
}

// The four cell tables in one: the queries' (points and edges, by their boxes
// inflated by dhat), then the primitives' (triangles and edges), table t's
// cells at t ncell.  A launch's workgroups go through the points, the edges
// as queries, the triangles and the edges as primitives; this is a lane's
// item: its table, its number and the cells it covers.  One launch and one scan
// per step for all tables: on small scenes, which are bound by launches,
// 19 fewer of 48 (two 16 x 16 sheets, a Newton step: 725 -> 655 us; three
// 101 x 101: 1250 -> 1150 us).
struct Item {
    int table;
    int64_t i;
    bool valid;
    int lo[3], hi[3];
};

__device__ __forceinline__ Item item_cells(const double* __restrict__ X, int64_t V, const Prims& pr,
                                           const PrimRec* __restrict__ erec, const Grid& g, double dhat) {
    Item it;
    const int64_t n[4] = {V, pr.E, pr.F, pr.E};
    int64_t b = blockIdx.x;
    it.table = 0;
    while (it.table < 3 && b >= blocks_of(n[it.table])) b -= blocks_of(n[it.table++]);
    const int64_t i = b * kBlock + threadIdx.x;
    it.valid = i < n[it.table];
    it.i = it.valid ? i : 0;
    Box box;
    if (it.table == 0) {
        box.lo = box.hi = ld3(X, (int)it.i);
    } else if (it.table == 2) {
        box = prim_box(X, pr.tris + 3 * it.i, 3);
    } else {
        const PrimRec& r = erec[it.i];
        box.lo = mk(r.lo[0], r.lo[1], r.lo[2]);
        box.hi = mk(r.hi[0], r.hi[1], r.hi[2]);
    }
    query_cells(box, g, it.table < 2 ? dhat : 0.0, it.lo, it.hi);
    return it;
}

// count[table ncell + cell] += items covering the cell; span[query] = cells
// the query covers (points first, then edges)
__global__ void __launch_bounds__(kBlock) k_cells_count(const double* __restrict__ X, int64_t V, Prims pr,
                                                        const PrimRec* __restrict__ erec, Grid g, double dhat,
                                                        int32_t* __restrict__ span, int32_t* __restrict__ count) {
    __shared__ uint32_t tab[kBlock / 64][kGroupSlots];
    const Item it = item_cells(X, V, pr, erec, g, dhat);
    if (it.valid && it.table < 2)
        span[(it.table ? V : 0) + it.i] =
            (it.hi[0] - it.lo[0] + 1) * (it.hi[1] - it.lo[1] + 1) * (it.hi[2] - it.lo[2] + 1);
    count += it.table * ((int64_t)g.n[0] * g.n[1] * g.n[2]);
    const auto vcell = [&](int a, int c, int e) { return ((int64_t)a * g.n[1] + c) * g.n[2] + e; };
    wave_visits(it.lo, it.hi, it.valid, (int32_t)it.i, vcell,
                [&](int64_t cell, int32_t, bool there) { count_visit(cell, there, count, tab[threadIdx.x >> 6]); });
}

// the items covering each cell, in no particular order: queries into ent
// (output positions come from the query and the cell, not from this order),
// primitives into raw, which lacks the queries' part
__global__ void __launch_bounds__(kBlock) k_cells_fill(const double* __restrict__ X, int64_t V, Prims pr,
                                                       const PrimRec* __restrict__ erec, Grid g, double dhat,
                                                       const int64_t* __restrict__ off, int32_t* __restrict__ fill,
                                                       int32_t* __restrict__ raw, int32_t* __restrict__ ent) {
    __shared__ uint32_t tab[kBlock / 64][kGroupSlots];
    const Item it = item_cells(X, V, pr, erec, g, dhat);
    const int64_t ncell = (int64_t)g.n[0] * g.n[1] * g.n[2];
    int32_t* to = it.table < 2 ? ent : raw - off[2 * ncell];
    off += it.table * ncell;
    fill += it.table * ncell;
    const auto vcell = [&](int a, int c, int e) { return ((int64_t)a * g.n[1] + c) * g.n[2] + e; };
    wave_visits(it.lo, it.hi, it.valid, (int32_t)it.i, vcell, [&](int64_t cell, int32_t item, bool there) {
        fill_visit(cell, item, there, off, fill, to, tab[threadIdx.x >> 6]);
    });
}

// each cell's list in increasing primitive id, one wave per cell: an entry's
// place is the number of entries of the cell below it (the ids of a cell
// are distinct), counted against the others handed over by lane reads;
// raw (which starts at the first cell's entry) -> ent; ncell = cells of both
// primitive tables, c0 = the launch's first
__global__ void __launch_bounds__(kBlock) k_cell_sort(int64_t c0, int64_t ncell, const int64_t* __restrict__ off,
                                                      const int32_t* __restrict__ raw,
                                                      int32_t* __restrict__ ent) {
    const int lane = threadIdx.x & 63;
    const int64_t c =
        c0 + (int64_t)blockIdx.x * (kBlock / 64) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (c >= ncell) return;
    const int64_t b = off[c], n = off[c + 1] - b;
    raw -= off[0];
    for (int64_t m0 = 0; m0 < n; m0 += 64) {
        const bool mine_ok = m0 + lane < n;
        const int32_t mine = mine_ok ? raw[b + m0 + lane] : 0;
        int rank = 0;
        for (int64_t c1 = 0; c1 < n; c1 += 64) {
            const int32_t other = c1 + lane < n ? raw[b + c1 + lane] : 0;
            const int m = (int)(n - c1 < 64 ? n - c1 : 64);
            for (int k = 0; k < m; ++k) rank += __builtin_amdgcn_readlane(other, k) < mine;
        }
        if (mine_ok) ent[b + rank] = mine;
    }
}

// a lane's 64-bit value, read by every lane (k wave-uniform)
__device__ __forceinline__ unsigned long long read_lane_u64(unsigned long long v, int k) {
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)v, k);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(v >> 32), k);
    return ((unsigned long long)hi << 32) | lo;
}

// a lane's double, read by every lane (k wave-uniform)
__device__ __forceinline__ double read_lane(double v, int k) {
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)b, k);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), k);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

// Boxes in whole steps of 1/2048 cell about a cell's corner, for a first test
// that rejects a pair by integers: a coordinate goes to -16383 .. 16383 by
// operations that never swap two values, so integers in strict order prove the
// order of the values (equal ones prove nothing, and NaN goes to the end that
// rejects nothing, as a comparison with it does).  Two axis ends per word: a
// primitive holds (hi, -lo) and a query (lo - dhat, -(hi + dhat)); a negative
// half of their difference says that the boxes are apart.
struct CellSteps {
    double org[3], inv[3];
};

__device__ __forceinline__ CellSteps cell_steps(const Grid& g, const int cc[3]) {
    CellSteps c;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        c.org[d] = g.org[d] + cc[d] * g.h[d];
        c.inv[d] = 2048.0 * g.inv[d];
    }
    return c;
}

typedef short short2_t __attribute__((ext_vector_type(2)));

__device__ __forceinline__ int step_lo(double v, const CellSteps& c, int d) {
    return (int)fmin(fmax((v - c.org[d]) * c.inv[d], -16383.0), 16383.0);
}

__device__ __forceinline__ int step_hi(double v, const CellSteps& c, int d) {
    return (int)fmax(fmin((v - c.org[d]) * c.inv[d], 16383.0), -16383.0);
}

__device__ __forceinline__ int pack_steps(int a, int b) { return (a & 0xffff) | (b << 16); }

__device__ __forceinline__ short2_t gap_steps(int prim, int query) {
    return __builtin_bit_cast(short2_t, prim) - __builtin_bit_cast(short2_t, query);
}

__device__ __forceinline__ short2_t min_steps(short2_t a, short2_t b) { return __builtin_elementwise_min(a, b); }

__device__ __forceinline__ int neg_steps(short2_t a) { return __builtin_bit_cast(int, a) & (int)0x80008000; }

// the words of a primitive's box and of a query's (already inflated) box
__device__ __forceinline__ void prim_steps(const double* lo, const double* hi, const CellSteps& c, int w[3]) {
#pragma unroll
    for (int d = 0; d < 3; ++d) w[d] = pack_steps(step_hi(hi[d], c, d), -step_lo(lo[d], c, d));
}

__device__ __forceinline__ void query_steps(const double* lo, const double* hi, const CellSteps& c, int w[3]) {
#pragma unroll
    for (int d = 0; d < 3; ++d) w[d] = pack_steps(step_lo(lo[d], c, d), -step_hi(hi[d], c, d));
}

// Edge-edge pairs, one wave per cell: its lanes take the edge queries
// covering the cell, 64 at a time, and the cell's edge list 64 records at a
// time, one record per lane; each record is then handed to every lane from
// the lane holding it (a lane read, no memory access), so the records are
// read once, or once per 64 queries where there are more than 64 of them.
// The query q's visit of the cell is entry e = qeoff[q] + j, j the cell's
// rank in the query's walk (x slowest, z fastest): EMIT = false stores the
// entry's candidate count in cnt[e], EMIT = true writes its candidates at
// out + eoff[e], in list order.  Only edges of larger index
// than the query are taken.  The counting pass also stores, per record
// and chunk of queries, the 64-lane mask of the queries it pairs with
// (bal, from boff[cell]); the emitting pass replays those masks instead of
// testing again, reading only the edges' vertex ids, and writes query by
// query so that a store covers consecutive slots of one query.  The
// counting pass also leaves each visit's entry e in evis (by position in
// the cell's query list), so the emitting pass needs no query boxes.
//
// The cell reporting a pair holds the lower corner of the overlap, whose
// coordinate along d is the larger of the inflated query's and the
// primitive's lower bounds; the cell index is monotonic in the coordinate,
// so that cell is, per axis, the larger of the two lower bounds' cells, and
// both are at most the current cell's (both boxes cover it): the pair is
// this cell's when, along every axis, one of the two lower cells is this
// cell's.
//
// The counting pass is bound by its instructions: some 24 records against 64
// queries a wave, 9 pairs in 100 a hit, so an early way out of the test is
// worth nothing (6%); integer steps with the coordinates looked at only for
// ties, one cell's setup without 64-bit divisions and with a reciprocal, and
// short lists kept for all queries took it from 956 to 690 us on ten
// 256 x 256 sheets (the point-triangle pass below from 461 to 310).  The
// emitting pass is bound by the lines it touches: the vertex ids come from the
// edges and not from the records, and consecutive cells share an L2 (613 ->
// 550 us; writing record by record, each query's lane its own slot, took 750).
// Six waves per SIMD: seven leave the counting pass 72 registers, ten spilled.
template <bool EMIT>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(6))) k_cell_pairs_ee(
                                                       const double* __restrict__ X,
                                                       const int32_t* __restrict__ vobj,
                                                       const PrimRec* __restrict__ erec,
                                                       const int32_t* __restrict__ edges, Grid g, double dhat,
                                                       int64_t c0, int64_t ncell, const int64_t* __restrict__ qtoff,
                                                       const int32_t* __restrict__ qent,
                                                       const int64_t* __restrict__ qeoff,
                                                       const int64_t* __restrict__ coff,
                                                       const int32_t* __restrict__ cent, int32_t* __restrict__ cnt,
                                                       const int64_t* __restrict__ eoff,
                                                       const int64_t* __restrict__ boff,
                                                       unsigned long long* __restrict__ bal,
                                                       int64_t* __restrict__ evis, int4* __restrict__ out) {
    const int lane = threadIdx.x & 63;
    const int64_t cell =
        c0 + xcd_block() * (kBlock / 64) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (cell >= ncell) return;
    const int64_t qa = qtoff[cell], qz = qtoff[cell + 1];
    const int64_t ta = coff[cell], tz = coff[cell + 1];
    if (qa == qz || (EMIT && ta == tz)) return;
    const uint32_t row = (uint32_t)cell / (uint32_t)g.n[2];  // at most 2^28 cells
    const int cc[3] = {(int)(row / (uint32_t)g.n[1]), (int)(row % (uint32_t)g.n[1]),
                       (int)((uint32_t)cell - row * (uint32_t)g.n[2])};
    const CellSteps st = cell_steps(g, cc);
    // the records in the lanes, those of the cell's first 64 on their way
    // beside the first queries; a short list stays for all queries
    int64_t at = ta;
    const int64_t bcell = boff[cell];
    int32_t id = 0;
    PrimRec r{};
    const auto load = [&](PrimRec& r) {
        if (EMIT) {
            r.v[0] = edges[2 * (int64_t)id];
            r.v[1] = edges[2 * (int64_t)id + 1];
        } else {
            r = erec[id];
        }
    };
    if (ta < tz) {
        id = cent[ta + lane < tz ? ta + lane : ta];
        load(r);
    }
    for (int64_t qb0 = qa; qb0 < qz; qb0 += 64) {
        const int64_t i = qb0 + lane;
        const bool act = i < qz;
        const int64_t q = qent[act ? i : qa];
        Box qb{};
        int32_t q0 = 0, q1 = 0, qo = 0;
        bool mixed = false;
        int lo[3] = {0, 0, 0}, hi[3] = {0, 0, 0};
        int64_t e, w = 0, wz = 0;
        if (EMIT) {
            // the counting pass left the visit's entry; only the query's ids
            // are needed
            e = act ? evis[i] : 0;
            q0 = edges[2 * q];
            q1 = edges[2 * q + 1];
            w = act ? eoff[e] : 0;
            wz = act ? eoff[e + 1] : 0;
            if (__ballot(w < wz) == 0) continue;
        } else {
            query_of<1>(q, X, vobj, erec, qb, q0, q1, qo);
            mixed = erec[q].v[2] != 0;
            query_cells(qb, g, dhat, lo, hi);
            e = qeoff[q] + ((int64_t)(cc[0] - lo[0]) * (hi[1] - lo[1] + 1) + (cc[1] - lo[1])) *
                               (hi[2] - lo[2] + 1) + (cc[2] - lo[2]);
            if (act) evis[i] = e;
        }
        const bool own0 = lo[0] == cc[0], own1 = lo[1] == cc[1], own2 = lo[2] == cc[2];
        const double qlx = qb.lo.x - dhat, qly = qb.lo.y - dhat, qlz = qb.lo.z - dhat;
        const double qhx = qb.hi.x + dhat, qhy = qb.hi.y + dhat, qhz = qb.hi.z + dhat;
        int qw[3] = {0, 0, 0};
        if (!EMIT) {
            const double ql[3] = {qlx, qly, qlz}, qh[3] = {qhx, qhy, qhz};
            query_steps(ql, qh, st, qw);
        }
        // axes whose lower cell is not this one, bit 3: no query
        const int qno = (own0 ? 0 : 1) | (own1 ? 0 : 2) | (own2 ? 0 : 4) | (act ? 0 : 8);
        const int32_t qid = (int32_t)q;
        // the list is in increasing edge id: skip what no lane takes
        int32_t qmin = act ? (int32_t)q : INT32_MAX;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) qmin = min(qmin, __shfl_xor(qmin, o, 64));
        qmin = __builtin_amdgcn_readfirstlane(qmin);
        int32_t found = 0;
        // this chunk's hit masks: slot (chunk of queries, record) of the cell
        const int64_t bslot = bcell + ((qb0 - qa) >> 6) * (tz - ta);
        for (int64_t tb0 = ta; tb0 < tz; tb0 += 64) {
            const int nk = (int)(tz - tb0 < 64 ? tz - tb0 : 64);
            if (at != tb0) {
                at = tb0;
                id = cent[tb0 + (lane < nk ? lane : 0)];
                load(r);
            }
            const int k0 = __popcll(__ballot(lane < nk && id <= qmin));
            if (k0 == nk) continue;
            if (EMIT) {
                // replay the counting pass's masks, query by query (only
                // the queries with a hit in this chunk): the hit records'
                // lanes write the query's next candidates side by side
                const unsigned long long mine = lane < nk ? bal[bslot + (tb0 - ta) + lane] : 0ull;
                unsigned long long any = mine;
#pragma unroll
                for (int o = 32; o > 0; o >>= 1) any |= __shfl_xor(any, o, 64);
                any = read_lane_u64(any, 0);
                const unsigned long long below = (1ull << lane) - 1ull;
                while (any) {
                    const int jq = __builtin_ctzll(any);
                    any &= any - 1ull;
                    const bool bit = (mine >> jq) & 1ull;
                    const unsigned long long bm = __ballot(bit);
                    const int64_t base = (int64_t)read_lane_u64((unsigned long long)w, jq);
                    const int32_t a0 = __builtin_amdgcn_readlane(q0, jq), a1 = __builtin_amdgcn_readlane(q1, jq);
                    if (bit)
                        out[base + __popcll(bm & below)] =
                            make_int4(a0, a1, r.v[0], r.v[1]);
                    if (lane == jq) w += __popcll(bm);
                }
                if (__ballot(w < wz) == 0) break;
                continue;
            }
            int tno = 8;  // as qno, bit 3 always
#pragma unroll
            for (int d = 0; d < 3; ++d)
                tno |= (cell_of(r.lo[d], g, d) != cc[d]) << d;
            int tw[3];
            prim_steps(r.lo, r.hi, st, tw);
            // ends of different objects: two edges of different objects may
            // share a vertex
            const unsigned long long share = __ballot((lane < nk && r.v[2] != 0) || mixed) ? ~0ull : 0ull;
            unsigned long long mine = 0;
            for (int k = k0; k < nk; ++k) {
                const short2_t gap =
                    min_steps(min_steps(gap_steps(__builtin_amdgcn_readlane(tw[0], k), qw[0]),
                                        gap_steps(__builtin_amdgcn_readlane(tw[1], k), qw[1])),
                              gap_steps(__builtin_amdgcn_readlane(tw[2], k), qw[2]));
                // wave masks: not apart and reported here, other object, later edge
                unsigned long long m =
                    __ballot((neg_steps(gap) | (__builtin_amdgcn_readlane(tno, k) & qno)) == 0) &
                    __ballot(__builtin_amdgcn_readlane(r.obj, k) != qo) &
                    __ballot(__builtin_amdgcn_readlane(id, k) > qid);
                const unsigned long long tie = __ballot(neg_steps(gap - (short)1) != 0);
                if ((m & (tie | share)) != 0ull) {
                    const double lx = read_lane(r.lo[0], k), ly = read_lane(r.lo[1], k), lz = read_lane(r.lo[2], k);
                    const double hx = read_lane(r.hi[0], k), hy = read_lane(r.hi[1], k), hz = read_lane(r.hi[2], k);
                    const int32_t v0 = __builtin_amdgcn_readlane(r.v[0], k), v1 = __builtin_amdgcn_readlane(r.v[1], k);
                    m &= ~__ballot(v0 == q0 || v0 == q1 || v1 == q0 || v1 == q1 || qlx > hx || lx > qhx || qly > hy ||
                                   ly > qhy || qlz > hz || lz > qhz);
                }
                if (lane == k) mine = m;
                found += __builtin_amdgcn_inverse_ballot_w64(m) ? 1 : 0;
            }
            if (lane < nk) bal[bslot + (tb0 - ta) + lane] = mine;
        }
        if (!EMIT && act) cnt[e] = found;
    }
}

// Point-triangle pairs of a cell the other way round: the cell's triangles
// in the lanes, 64 at a time, and its points (a cell holds tens of them,
// fewer than triangles) handed to every lane by lane reads, so a wave step
// tests one point against 64 triangles.  The points' setup (entry e,
// reporting-cell flags) is done with the points in the lanes, 64 at a
// time.  A pair is taken when the point and the triangle belong to
// different objects, the point is none of the triangle's vertices, the
// point's box inflated by dhat overlaps the triangle's box and the cell
// reports it (as for the edges); the counting pass stores each point's
// 64-bit mask over a chunk of triangles at bal + boff[cell] + (triangle
// chunk) * (points of the cell) + (point's place in the cell's list), and
// the emitting pass replays them, writing at out + eoff[e] in list order.
template <bool EMIT>
__global__ void __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(7)))
k_cell_pairs_pt(const double* __restrict__ X, const int32_t* __restrict__ vobj, const PrimRec* __restrict__ trec,
                const int32_t* __restrict__ tris, Grid g, double dhat, int64_t c0, int64_t ncell, const int64_t* __restrict__ qtoff,
                const int32_t* __restrict__ qent, const int64_t* __restrict__ qeoff,
                const int64_t* __restrict__ coff, const int32_t* __restrict__ cent, int32_t* __restrict__ cnt,
                const int64_t* __restrict__ eoff, const int64_t* __restrict__ boff,
                unsigned long long* __restrict__ bal, int64_t* __restrict__ evis, int4* __restrict__ out) {
    const int lane = threadIdx.x & 63;
    const int64_t cell =
        c0 + (int64_t)blockIdx.x * (kBlock / 64) + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (cell >= ncell) return;
    const int64_t qa = qtoff[cell], qz = qtoff[cell + 1];
    const int64_t ta = coff[cell], tz = coff[cell + 1];
    if (qa == qz || (EMIT && ta == tz)) return;
    const uint32_t row = (uint32_t)cell / (uint32_t)g.n[2];  // at most 2^28 cells
    const int cc[3] = {(int)(row / (uint32_t)g.n[1]), (int)(row % (uint32_t)g.n[1]),
                       (int)((uint32_t)cell - row * (uint32_t)g.n[2])};
    const CellSteps st = cell_steps(g, cc);
    const int64_t nq = qz - qa;
    const unsigned long long below = (1ull << lane) - 1ull;
    for (int64_t qb0 = qa; qb0 < qz; qb0 += 64) {
        const int64_t i = qb0 + lane;
        const bool act = i < qz;
        const int32_t q = qent[act ? i : qa];
        const int nqk = (int)(qz - qb0 < 64 ? qz - qb0 : 64);
        d3 pq = mk(0.0, 0.0, 0.0);
        int32_t qo = 0, qno = 0;
        int qw[3] = {0, 0, 0};
        int64_t e, w = 0, wz = 0;
        if (EMIT) {
            e = act ? evis[i] : 0;
            w = act ? eoff[e] : 0;
            wz = act ? eoff[e + 1] : 0;
            if (__ballot(w < wz) == 0) continue;
        } else {
            Box qb;
            int32_t q0, q1;
            query_of<0>(q, X, vobj, nullptr, qb, q0, q1, qo);
            pq = qb.lo;
            int lo[3], hi[3];
            query_cells(qb, g, dhat, lo, hi);
            e = qeoff[q] + ((int64_t)(cc[0] - lo[0]) * (hi[1] - lo[1] + 1) + (cc[1] - lo[1])) *
                               (hi[2] - lo[2] + 1) + (cc[2] - lo[2]);
            if (act) evis[i] = e;
            // axes whose lower cell is not this one, bit 3 always
            qno = (lo[0] != cc[0]) | ((lo[1] != cc[1]) << 1) | ((lo[2] != cc[2]) << 2) | 8;
            const double ql[3] = {pq.x - dhat, pq.y - dhat, pq.z - dhat};
            const double qh[3] = {pq.x + dhat, pq.y + dhat, pq.z + dhat};
            query_steps(ql, qh, st, qw);
        }
        int32_t found = 0;
        for (int64_t tb0 = ta; tb0 < tz; tb0 += 64) {
            const int64_t j = tb0 + lane;
            const bool tact = j < tz;
            const int32_t id = cent[tact ? j : tb0];
            const int64_t slot = boff[cell] + ((tb0 - ta) >> 6) * nq + (qb0 - qa);
            if (EMIT) {
                const int32_t* rv = tris + 3 * (int64_t)id;
                const int32_t r0 = rv[0], r1 = rv[1], r2 = rv[2];
                const unsigned long long mq = lane < nqk ? bal[slot + lane] : 0ull;
                for (int k = 0; k < nqk; ++k) {
                    const unsigned long long m = read_lane_u64(mq, k);
                    if (m == 0) continue;
                    const int64_t base = (int64_t)read_lane_u64((unsigned long long)w, k);
                    const int32_t a0 = __builtin_amdgcn_readlane(q, k);
                    if ((m >> lane) & 1ull) out[base + __popcll(m & below)] = make_int4(-(a0 + 1), r0, r1, r2);
                    if (lane == k) w += __popcll(m);
                }
                if (__ballot(w < wz) == 0) break;
                continue;
            }
            PrimRec r = trec[id];
            // vertices of different objects: a point of another object than
            // the first vertex's may be one of the others
            const unsigned long long share = __ballot(tact && r.v[2] < 0) ? ~0ull : 0ull;
            r.v[2] = r.v[2] < 0 ? ~r.v[2] : r.v[2];
            int tno = tact ? 0 : 8;  // as qno, bit 3: no triangle
#pragma unroll
            for (int d = 0; d < 3; ++d)
                tno |= (cell_of(r.lo[d], g, d) != cc[d]) << d;
            int tw[3];
            prim_steps(r.lo, r.hi, st, tw);
            unsigned long long mine = 0;
            for (int k = 0; k < nqk; ++k) {
                const short2_t gap =
                    min_steps(min_steps(gap_steps(tw[0], __builtin_amdgcn_readlane(qw[0], k)),
                                        gap_steps(tw[1], __builtin_amdgcn_readlane(qw[1], k))),
                              gap_steps(tw[2], __builtin_amdgcn_readlane(qw[2], k)));
                unsigned long long m =
                    __ballot((neg_steps(gap) | (__builtin_amdgcn_readlane(qno, k) & tno)) == 0) &
                    __ballot(__builtin_amdgcn_readlane(qo, k) != r.obj);
                const unsigned long long tie = __ballot(neg_steps(gap - (short)1) != 0);
                if ((m & (tie | share)) != 0ull) {
                    const double px = read_lane(pq.x, k), py = read_lane(pq.y, k), pz = read_lane(pq.z, k);
                    const int32_t a0 = __builtin_amdgcn_readlane(q, k);
                    m &= ~__ballot(r.v[0] == a0 || r.v[1] == a0 || r.v[2] == a0 || px - dhat > r.hi[0] ||
                                   r.lo[0] > px + dhat || py - dhat > r.hi[1] || r.lo[1] > py + dhat ||
                                   pz - dhat > r.hi[2] || r.lo[2] > pz + dhat);
                }
                if (lane == k) {
                    mine = m;
                    found += __popcll(m);
                }
            }
            if (lane < nqk) bal[slot + lane] = mine;
        }
        if (!EMIT && act) cnt[e] = found;
    }
}

// per cell, the hit-mask slots of its pairs passes: of the point-triangle
// pass (one per chunk of 64 triangles and point of the cell) at c, of the
// edge-edge pass (one per chunk of 64 queries and edge) at ncell + c
__global__ void __launch_bounds__(kBlock) k_cell_slots(int64_t ncell, const int64_t* __restrict__ off,
                                                       int64_t* __restrict__ n) {
    const int64_t c = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (c >= 2 * ncell) return;
    const int64_t nq = off[c + 1] - off[c], nt = off[2 * ncell + c + 1] - off[2 * ncell + c];
    n[c] = c < ncell ? ((nt + 63) >> 6) * nq : ((nq + 63) >> 6) * nt;
}

// The passes with one wavefront per cell run in slices of kCellSlice cells: a
// launch takes fewer than 2^32 work-items, which is 2^26 cells, and there are
// up to 2^28 in a grid and twice as many in the two primitive tables.
// launch(first cell, workgroups) for every slice of n cells.
constexpr int64_t kCellSlice = int64_t(1) << 25;
template <typename L>
hipError_t cell_slices(int64_t n, L launch) {
    for (int64_t c0 = 0; c0 < n; c0 += kCellSlice) {
        const int64_t m = n - c0 < kCellSlice ? n - c0 : kCellSlice;
        launch(c0, (unsigned)((m + kBlock / 64 - 1) / (kBlock / 64)));
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

Grid to_grid(const CandGrid& cg) {
    Grid g;
    for (int d = 0; d < 3; ++d) { g.org[d] = cg.org[d]; g.n[d] = cg.n[d]; g.h[d] = cg.h[d]; g.inv[d] = 1.0 / cg.h[d];
        if (!std::isfinite(g.inv[d])) g.inv[d] = 0.0;  // every test then falls back to the division
    }
    return g;
}

}  // namespace

int32_t cand_bound_blocks(int64_t V, int64_t FE) {
    const int64_t n = V > FE ? V : FE;
    int64_t b = (n + kBlock - 1) / kBlock;
    return (int32_t)(b < 1 ? 1 : (b > 1024 ? 1024 : b));
}

hipError_t launch_cand_bounds(const double* x, int32_t V, const int32_t* tris, int64_t F, const int32_t* edges,
                              int64_t E, CandBounds* part, int32_t nb, hipStream_t s) {
    k_cand_bounds<<<(unsigned)nb, kBlock, 0, s>>>(x, V, Prims{tris, edges, F, E}, part);
    return hipGetLastError();
}

hipError_t launch_prim_records(const double* x, const int32_t* tris, int64_t F, const int32_t* edges, int64_t E,
                               const int32_t* vobj, void* trec, void* erec, hipStream_t s) {
    const int64_t nb = blocks_of(F) + blocks_of(E);
    if (nb == 0) return hipSuccess;
    k_prim_records<<<(unsigned)nb, kBlock, 0, s>>>(x, Prims{tris, edges, F, E}, vobj, static_cast<PrimRec*>(trec),
                                                   static_cast<PrimRec*>(erec));
    return hipGetLastError();
}

hipError_t launch_cells_count(const double* x, int32_t V, const int32_t* tris, int64_t F, const int32_t* edges,
                              int64_t E, const void* erec, const CandGrid& cg, double dhat, int32_t* span,
                              int32_t* count, hipStream_t s) {
    const int64_t nb = blocks_of(V) + blocks_of(F) + 2 * blocks_of(E);
    if (nb == 0) return hipSuccess;
    k_cells_count<<<(unsigned)nb, kBlock, 0, s>>>(x, V, Prims{tris, edges, F, E}, static_cast<const PrimRec*>(erec),
                                                  to_grid(cg), dhat, span, count);
    return hipGetLastError();
}

hipError_t launch_cells_fill(const double* x, int32_t V, const int32_t* tris, int64_t F, const int32_t* edges,
                             int64_t E, const void* erec, const CandGrid& cg, double dhat, const int64_t* off,
                             int32_t* fill, int32_t* raw, int32_t* ent, hipStream_t s) {
    const Grid g = to_grid(cg);
    const int64_t ncell = (int64_t)g.n[0] * g.n[1] * g.n[2];
    const int64_t nb = blocks_of(V) + blocks_of(F) + 2 * blocks_of(E);
    if (nb == 0) return hipSuccess;
    k_cells_fill<<<(unsigned)nb, kBlock, 0, s>>>(x, V, Prims{tris, edges, F, E}, static_cast<const PrimRec*>(erec),
                                                 g, dhat, off, fill, raw, ent);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    return cell_slices(2 * ncell, [&](int64_t c0, unsigned nwg) {
        k_cell_sort<<<nwg, kBlock, 0, s>>>(c0, 2 * ncell, off + 2 * ncell, raw, ent);
    });
}

hipError_t launch_cell_slots(const CandGrid& cg, const int64_t* off, int64_t* n, hipStream_t s) {
    const int64_t ncell = (int64_t)cg.n[0] * cg.n[1] * cg.n[2];
    k_cell_slots<<<(unsigned)blocks_of(2 * ncell), kBlock, 0, s>>>(ncell, off, n);
    return hipGetLastError();
}

hipError_t launch_cell_pairs(int kind, bool emit, const double* x, const int32_t* vobj, const int32_t* prims,
                             const void* rec, const CandGrid& cg, double dhat, const int64_t* qtoff,
                             const int32_t* qent, const int64_t* qeoff, const int64_t* coff, const int32_t* cent,
                             int32_t* cnt, const int64_t* eoff, const int64_t* boff, uint64_t* bal,
                             int64_t* evis, int32_t* out, hipStream_t s) {
    const Grid g = to_grid(cg);
    const int64_t ncell = (int64_t)g.n[0] * g.n[1] * g.n[2];
    int4* o = reinterpret_cast<int4*>(out);
    const PrimRec* pr = static_cast<const PrimRec*>(rec);
    unsigned long long* b = reinterpret_cast<unsigned long long*>(bal);
    const auto kernel = kind == 0 ? (emit ? k_cell_pairs_pt<true> : k_cell_pairs_pt<false>)
                                  : (emit ? k_cell_pairs_ee<true> : k_cell_pairs_ee<false>);
    return cell_slices(ncell, [&](int64_t c0, unsigned nwg) {
        kernel<<<nwg, kBlock, 0, s>>>(x, vobj, pr, prims, g, dhat, c0, ncell, qtoff, qent, qeoff, coff, cent, cnt, eoff,
                                      boff, b, evis, o);
    });
}

}  // namespace gipc
