// Host-side internals shared by the translation units of libgipc: the
// context, device buffers and the kernel launchers each .hip file provides.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>
#include <utility>
#include <vector>

#include "../../include/gipc.h"
#include "device_math.hpp"

namespace gipc {

constexpr int kBlock = 256;          // threads per workgroup (4 waves of 64)
constexpr int kScanItems = 8;        // elements per thread in the scans
constexpr int kMaxRowPairs = 2048;   // pairs touching one vertex (LDS sort capacity, 64 KiB)
// Vertices per energy piece.  The sum over one is a chain of loads of its
// workgroup: five 150 x 150 sheets 4.9 us at 1024, 15.8 us at 8192 (14 pieces);
// shorter pieces only lengthen the sum over a scene's pieces.
constexpr int kEnergyPiece = 1024;

// Grow-only device buffer, from hipMalloc or from the caller's allocator
// (al non-null; device = the context's device).
struct DevBuf {
    void* p = nullptr;
    size_t bytes = 0;
    const gipc_allocator* al = nullptr;
    int device = 0;
};

hipError_t ensure(DevBuf& b, size_t bytes);
void release(DevBuf& b);

template <typename T>
inline T* as(DevBuf& b) { return static_cast<T*>(b.p); }

// Workgroups go to the chip's 8 XCDs in turn (workgroup b runs on XCD
// b mod 8), and every XCD has an L2 of its own.  xcd_run() renumbers a launch
// of n workgroups, 8 RUN at a time, so that each XCD takes a run of RUN
// neighbouring ones: the neighbouring rows of a gather kernel then
// read the records they share through the same L2.  It is a permutation of
// 0 .. n-1.  One run per XCD over the whole launch left XCDs waiting
// where work is uneven and spread the traffic over eight places of every
// array (assembly of 64 scenes of 32^2 to 256^2 vertices 7200 us, of ten
// 256 x 256 sheets 2885); runs of 256 take 6360 and 2832, of 1024 6390 and
// 2850, of 32 6470 and 2935, of 8 6760 and 3080.
constexpr int kXcds = 8, kXcdRun = 256;
template <int RUN = kXcdRun>
__device__ __forceinline__ uint32_t xcd_run(uint32_t b, uint32_t n) {
    constexpr uint32_t turn = kXcds * RUN;
    const uint32_t base = b / turn * turn;
    const uint32_t m = n - base < turn ? n - base : turn;  // workgroups of this turn
    const uint32_t q = m / kXcds, r = m % kXcds, i = b - base, x = i % kXcds;
    return base + x * q + (x < r ? x : r) + i / kXcds;
}

__device__ __forceinline__ int64_t xcd_block() { return (int64_t)xcd_run(blockIdx.x, gridDim.x); }

// Ranges of staged pairs per sub-type: pairs of type t occupy [off[t], off[t+1]).
struct TypeRanges {
    int64_t off[9];
};

__device__ __forceinline__ int type_of(int64_t k, const TypeRanges& tr) {
    int t = 1;
    while (t < 7 && k >= tr.off[t + 1]) ++t;
    return t;
}

__device__ __forceinline__ int vslot(const int4& v, int j) {
    return j == 0 ? v.x : (j == 1 ? v.y : (j == 2 ? v.z : v.w));
}

__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int D>
__device__ __forceinline__ double quad_xor(double v) {  // the value of lane ^ D, D = 1 or 2
    constexpr int ctrl = D == 1 ? 0xB1 : 0x4E;           // quad_perm [1,0,3,2], [2,3,0,1]
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_mov_dpp((int)b, ctrl, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), ctrl, 0xF, 0xF, false);
    return __longlong_as_double(((long long)hi << 32) | (long long)(unsigned)lo);
}

template <int D>
__device__ __forceinline__ void quad_swap(double2& a, double2& b, bool odd) {
    const double2 s = odd ? a : b;
    const double2 r = make_double2(quad_xor<D>(s.x), quad_xor<D>(s.y));
    if (odd) a = r;
    else b = r;
}

// element t of lane p becomes element p of lane t
__device__ __forceinline__ void quad_transpose(double2 (&v)[4]) {
    const bool p1 = threadIdx.x & 1, p2 = threadIdx.x & 2;
    quad_swap<1>(v[0], v[1], p1);
    quad_swap<1>(v[2], v[3], p1);
    quad_swap<2>(v[0], v[2], p2);
    quad_swap<2>(v[1], v[3], p2);
}

template <int T>
__device__ __forceinline__ uint32_t quad_lane(uint32_t v) {  // the value of the quad's lane T
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, 0x55 * T, 0xF, 0xF, false);
}

// Writes 64-byte records, one per lane, a quad of lanes at a time: after a
// transpose within the quad each of four steps writes one record whole, 16
// bytes per lane, so an instruction touches 16 lines and not 64.  All four
// lanes of a quad must be active; record ~0u: none.  Loading records the same
// way did not pay (ten 256 x 256 sheets: both assembly passes within 5%).
__device__ __forceinline__ void quad_store(double* __restrict__ base, uint32_t rec, double2 (&v)[4]) {
    double2* b = reinterpret_cast<double2*>(base) + (threadIdx.x & 3);
    const uint32_t k[4] = {quad_lane<0>(rec), quad_lane<1>(rec), quad_lane<2>(rec), quad_lane<3>(rec)};
    quad_transpose(v);
#pragma unroll
    for (int t = 0; t < 4; ++t)
        if (k[t] != ~0u) b[4 * (int64_t)k[t]] = v[t];
}

// Groups of equal keys among the lanes of a wavefront, wherever they sit: a
// group's leader is its lowest lane, rank numbers its lanes from 0 (in no
// particular order), count is its size.  One atomic per group then replaces
// one per lane.  Each round the open lanes meet in an LDS table of 128 slots
// at the hash of their key, where the lowest lane wins; lanes with the
// winner's key are done, the others meet again under another hash.  With some
// 25 distinct keys in a wavefront that is about two rounds of 25
// instructions, where one round per distinct key took 25 rounds of 15.
// tab: 128 words of LDS of this wavefront alone.
constexpr int kGroupSlots = 128;

struct WaveGroup {
    int leader, rank, count;  // leader -1 for lanes not in
};

template <int N>
__device__ __forceinline__ WaveGroup wave_group(const int (&key)[N], bool in, uint32_t* tab) {
    const int lane = threadIdx.x & 63;
    WaveGroup g{-1, 0, 0};
    uint32_t h = 0u;
#pragma unroll
    for (int n = 0; n < N; ++n) h = (h ^ (uint32_t)key[n]) * 0x9e3779b1u;
    h ^= h >> 15;
    bool open = in;
    while (__ballot(open) != 0ull) {
        tab[lane] = ~0u;
        tab[lane + 64] = ~0u;
        wave_lds_fence();
        if (open) atomicMin(&tab[h % kGroupSlots], (uint32_t)lane);
        wave_lds_fence();
        const int w = open ? (int)tab[h % kGroupSlots] : lane;
        bool same = open;
#pragma unroll
        for (int n = 0; n < N; ++n) same = __shfl(key[n], w, 64) == key[n] && same;
        if (same) {
            g.leader = w;
            open = false;
        }
        h = (h >> 7) * 0x85ebca6bu + 1u;
        wave_lds_fence();
    }
    tab[lane] = 0u;
    wave_lds_fence();
    if (in) g.rank = (int)atomicAdd(&tab[g.leader], 1u);
    wave_lds_fence();
    if (in) g.count = (int)tab[g.leader];
    wave_lds_fence();
    return g;
}

// One tuple in the paper's sign encoding (Sec. 7.2, "Data structures"),
// negative ids as -(i+1), decoded with ~i:
//   [a0, a1, b0, b1]            edge-edge (a1 negative: close to parallel)
//   [-p, t0, t1, t2]            point-triangle
//   [-p, e0, e1, -1]            point-edge
//   [-p, q, -1, -1]             point-point
//   [-p, -o, e0, -e1]           point-edge cut from a close-to-parallel
//                               edge-edge pair (p's edge is (p, o))
//   [-p, -o, -q, -r]            point-point cut from one (q's edge is (q, r))
// Returns the kind (0 EE, 1 PT, 2 PE, 3 PP, 4 PE cut from EE, 5 PP cut
// from EE) with the vertex ids in v (nv of them), or -1 for a malformed
// tuple: a pattern not above, an id outside [0, V) or a repeated id.
__device__ __forceinline__ int decode_tuple(const int4 t, int32_t V, int v[4], int& nv) {
    int kind = -1;
    if ((t.z | t.w) >= 0 && (t.x & t.y) >= 0) {
        // the two kinds a broad phase gives, without the branches of the rest
        v[0] = t.x >= 0 ? t.x : ~t.x;
        v[1] = t.y >= 0 ? t.y : ~t.y;
        v[2] = t.z;
        v[3] = t.w;
        nv = 4;
        const bool ok = max(max(v[0], v[1]), max(v[2], v[3])) < V && v[0] != v[1] && v[0] != v[2] && v[0] != v[3] &&
                        v[1] != v[2] && v[1] != v[3] && v[2] != v[3];
        return ok ? (t.x >= 0 ? 0 : 1) : -1;
    }
    v[0] = v[1] = v[2] = v[3] = -1;
    nv = 0;
    if (t.x < 0 && t.y >= 0) {
        v[0] = ~t.x; v[1] = t.y;
        if (t.z >= 0 && t.w == -1) { kind = 2; nv = 3; v[2] = t.z; }
        else if (t.z == -1 && t.w == -1) { kind = 3; nv = 2; }
    } else if (t.x < 0 && t.w < 0) {
        v[0] = ~t.x; v[1] = ~t.y; v[3] = ~t.w; nv = 4;
        if (t.z >= 0) { kind = 4; v[2] = t.z; }
        else { kind = 5; v[2] = ~t.z; }
    }
    bool ok = kind >= 0;
    for (int k = 0; k < nv && ok; ++k) {
        ok = v[k] >= 0 && v[k] < V;
        for (int l = 0; l < k && ok; ++l) ok = v[l] != v[k];
    }
    return ok ? kind : -1;
}

// wave64 sum by a fixed butterfly, then the block's waves in order: the
// result does not depend on scheduling.  NT = threads of the workgroup.
template <int NT>
__device__ __forceinline__ double block_sum_n(double v, double* lds /*[NT/64]*/) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int w = 0; w < NT / 64; ++w) s += lds[w];
    __syncthreads();
    return s;  // valid in thread 0
}

__device__ __forceinline__ double block_sum(double v, double* lds /*[kBlock/64]*/) {
    return block_sum_n<kBlock>(v, lds);
}

struct PcgScalars {  // device-resident scalars of the PCG loop
    double rz, pq, rr, bb, alpha, beta, rtol2, rz0;
    int iters, done, breakdown, maxit;
    int delta;  // stopping test: 0 r.r <= rtol2 b.b, 1 r.z <= rtol2 r0.z0
    int conv;   // the stopping test held
    int stop;       // what the merged update found, for the p update
    double rzb[2];  // r.z by the parity of the iteration that reads it
};

}  // namespace gipc

struct gipc_ctx {
    int device = 0;
    std::string err;
    gipc_allocator alloc{};  // the caller's allocator (alloc.alloc null: hipMalloc)

    // staging (per candidate)
    gipc::DevBuf cand_ft, cand_vid, bcount, boff, counters;
    // staged pairs, sorted by sub-type; mult = multiplicity of merged
    // duplicates (valid when merged)
    gipc::DevBuf st_vid, st_src, mult;
    bool merged = false;
    // merge scratch
    gipc::DevBuf mkeys, mslots, mrep_of, mcount, mbcount, mpos, st_vid2, st_src2;
    gipc::TypeRanges ranges{};
    int64_t Ps = 0;
    int32_t V = 0;
    // symbolic
    gipc::DevBuf deg, kcount, fill, inc_ptr, kptr, contrib, kcol, kbeg, ncols, row_ptr, col_idx, cptr, slot_row,
        diag_slot, maxbuf, bigrows, tslot, incr;
    // per 64 blocks of the pattern: head bits of row starts, row of the first block
    gipc::DevBuf whead, wrow;
    // visiting order of the block rows in the assembly (spatial cells)
    gipc::DevBuf order, obox, ocell, ohist, ooff, ofill;
    int64_t nnzb = 0, K = 0;
    int32_t max_deg = 0;
    // scenes of the build: scene id per vertex (batches only), energy pieces
    // (vertex ranges of at most kEnergyPiece inside one scene) and the
    // scenes' piece offsets
    gipc::DevBuf vscene, pieces, poff;
    std::vector<int2> h_pieces;   // the tables pieces and poff hold
    std::vector<int32_t> h_poff;
    int32_t S = 1, npieces = 0;
    bool batched = false;
    // factors of the last eval; per-vertex energy shares and piece sums
    gipc::DevBuf rec_main, rec_extra, rec_a1, ev, epart;
    // matrix-free operator: the c_i w~_k vectors of every incidence, row by
    // row (built at the first use after an eval), and (alpha, beta) per pair
    gipc::DevBuf mfg, mfab;
    // lagged friction: per-pair lag and eval records, energy shares and
    // pieces; the build it was lagged for and eps_v dt
    gipc::DevBuf flag, ffr, fev, fpart;
    // contact candidates: bounds partials, counters, cell tables, primitive
    // records, per query its cells, per visit its candidates, hit masks
    gipc::DevBuf cpart, ccnt, ccount, cfill, coff, cent, craw, crec_t, crec_e, cspan, cqoff, ecnt, eoff, bslot, cboff,
        bal, evis;
    uint64_t fric_gen = 0;
    double fric_sv = 0.0;
    uint64_t eval_gen = 0;   // bumped by every eval
    uint64_t mfg_gen = 0;    // eval_gen the vectors in mfg belong to
    int64_t ninc = 0;  // incidences (k, i) of the build: sum of the stencil sizes
    // launch shapes (gipc_tune)
    gipc_tune tune{4, 16, 4, 0};
    // PCG workspace
    gipc::DevBuf r, z, p, q, p32, minv, part, scal;
    // scan scratch; counters of gipc_pairs_check
    gipc::DevBuf scan_tmp, scan_tmp2, chk;
    gipc::DevBuf accd_cnt;

    gipc_info info{};
    bool built = false;
    bool evaluated = false;
    uint64_t build_gen = 0;  // bumped by every gipc_pairs_build (graphs check it)
};

namespace gipc {

// ---- scan.hip
// out[i] = sum_{j<i} in[j] for i <= n (out has n+1 entries); *total_dev
// (device int64, nullable) receives the sum without narrowing.
// TIn: int32/int64, TOut: int32/int64.
template <typename TIn, typename TOut>
hipError_t exclusive_scan(const TIn* in, int64_t n, TOut* out, gipc_ctx* ctx, hipStream_t s,
                          int64_t* total_dev = nullptr);
// zeroes up to four int32 arrays in one launch and, with counters, sets its
// slots i < nslots to -1 where bit i of ones is set and to 0 otherwise
struct ZeroList {
    int32_t* p[4] = {nullptr, nullptr, nullptr, nullptr};
    int64_t n[4] = {0, 0, 0, 0};
};
hipError_t zero_i32(const ZeroList& z, hipStream_t s, int64_t* counters = nullptr, int nslots = 0,
                    uint64_t ones = 0);

// ---- stage.hip
hipError_t launch_vertex_scene(const int32_t* vert_off, int32_t S, int32_t V, int32_t* vscene, hipStream_t s);
hipError_t launch_stage_classify(const int32_t* tuples, int64_t P, int32_t V, const double* x, const double* xr,
                                 const DevParams& pm, uint8_t* ft, int4* vid, int32_t* bcount, int64_t* counters,
                                 hipStream_t s);
hipError_t launch_stage_scatter(const uint8_t* ft, const int4* vid, int64_t P, const int64_t* boff, int4* st_vid,
                                int32_t* st_src, int64_t* type_off, hipStream_t s);
// the build's classification (ft_b, vid_b) against the one at x; counters
// (device int64 [kCheckCopies][kCheckStride], each copy's first six zeroed,
// [5] = INT64_MAX): entered, left, changed, degenerate, malformed, first
// changed tuple; the result is the sum (the smallest [5]) over the copies in
// use, one per workgroup of kBlock tuples up to kCheckCopies
constexpr int kCheckCopies = 64, kCheckStride = 16;
hipError_t launch_stage_check(const int32_t* tuples, int64_t P, int32_t V, const double* x, const double* xr,
                              const DevParams& pm, const uint8_t* ft_b, const int4* vid_b, int64_t* counters,
                              hipStream_t s);

// ---- merge.hip
// merge duplicate PE / PP constraints of ctx->ranges (vertex ids < V) into
// one staged pair with a multiplicity (ctx->mult); swaps the staged arrays
// and writes the merged type offsets (9 int64) to new_off_dev
hipError_t merge_duplicates(gipc_ctx* ctx, int32_t V, hipStream_t s, int64_t* new_off_dev);

// ---- order.hip
// ctx->order = the vertices sorted into Morton cells of their bounding cube
// (scene-major with each scene's own cube when S > 1: vert_off device int32
// [S+1] and ctx->vscene must be set)
// row_order_tables first: its arrays, and in zero those that must be zeroed
hipError_t row_order_tables(gipc_ctx* ctx, int32_t V, int32_t S, ZeroList& zero, int at);
hipError_t build_row_order(gipc_ctx* ctx, const double* x, int32_t V, const int32_t* vert_off, int32_t S,
                           hipStream_t s);

// ---- symbolic.hip
// pairs touching each vertex (deg), their block contributions to its row
// (kcount) and the largest deg (max_deg, zero on entry); both: scratch, zero
// on entry; rank: each staged pair's place among its vertices' pairs, by slot
hipError_t launch_sym_count(const int4* st_vid, TypeRanges tr, int32_t V, unsigned long long* both, int4* rank,
                            int32_t* deg, int32_t* kcount, int32_t* max_deg, hipStream_t s);
// incr: one record per incidence: k << 2 | i, then the vertices of the pair's other
// slots in slot order (-1 past the stencil)
hipError_t launch_sym_scatter(const int4* st_vid, TypeRanges tr, const int64_t* inc_ptr, const int4* rank,
                              int4* incr, hipStream_t s);
// big: int32 [V] scratch for the rows sorted by whole workgroups, nbig: a
// device counter that must be zero on entry
// contrib: each row's sorted contribution codes; kcol / kbeg: the row's
// distinct columns and the offset of each one's first contribution, written
// compactly from the row's contribution offset; ncols: their count
hipError_t launch_sym_rowsort(int32_t V, int32_t max_deg, const int64_t* inc_ptr, const int4* incr,
                              TypeRanges tr, const int64_t* kptr, uint32_t* contrib,
                              int32_t* kcol, int32_t* kbeg, int32_t* ncols, int32_t* big, int64_t* nbig,
                              hipStream_t s);
hipError_t launch_sym_fill(int32_t V, const int64_t* kptr, const int32_t* kcol, const int32_t* kbeg,
                           const int32_t* row_ptr, int32_t* col_idx, int64_t* cptr, int32_t* slot_row,
                           int32_t* diag_slot, unsigned long long* whead, int32_t* wrow, int64_t nnzb,
                           hipStream_t s);
// tslot[s] = slot of (c, r) for every block s = (r, c) with c > r, else -1
hipError_t launch_sym_transpose(int64_t nnzb, const int32_t* slot_row, const int32_t* col_idx,
                                const int32_t* row_ptr, int32_t* tslot, hipStream_t s);

// ---- eval.hip
// waves: workgroup size in wavefronts (1, 2, 4 or 8)
// mult: multiplicity per staged pair, nullable (all 1)
hipError_t launch_eval(const int4* st_vid, const int32_t* mult, TypeRanges tr, const double* x, const double* xr,
                       const DevParams& pm, double* rec_main, double* rec_extra, double* rec_a1, int waves,
                       hipStream_t s);
// per-scene energies from the per-vertex shares: pieces, then scenes
hipError_t launch_energy(const double* ev, const int2* pieces, int32_t npieces, const int32_t* poff, int32_t S,
                         double* part, double* energy, hipStream_t s);

// ---- assemble.hip
// mode bit 1: gradient and per-vertex energy shares, bit 2: diagonal block
// values; lanes per row: 4, 8, 16 or 32
// rows are visited in the order `order` (a permutation of 0..V-1; null: 0..V-1)
hipError_t launch_rows_diag(int mode, int32_t V, const int32_t* order, const int32_t* diag_slot, const int64_t* cptr,
                            const uint32_t* contrib, const double* rec_main, const double* rec_extra,
                            const double* rec_a1, int64_t e0,
                            int64_t m0, const double* diag, double* grad, double* ev, void* val, int dtype,
                            int64_t nnzb, int lanes, hipStream_t s);
// blocks above the diagonal are summed once and stored with their
// transpose at tslot, row by row in the order `order` (null: storage order); waves: workgroup size
// in wavefronts (1, 2, 4 or 8)
hipError_t launch_offdiag(int32_t V, const int32_t* order, const int32_t* row_ptr, const int32_t* diag_slot,
                          int64_t nnzb, const int32_t* col_idx, const int32_t* tslot,
                          const int64_t* cptr, const uint32_t* contrib, const double* rec_main,
                          const double* rec_extra, int64_t e0, int64_t m0, void* val, int dtype, int waves,
                          hipStream_t s);
hipError_t launch_pair_inspect(const int4* st_vid, const int32_t* st_src, const int32_t* smult, TypeRanges tr,
                               const double* rec_main, const double* rec_extra, const double* rec_a1, const double* x,
                               const double* xr,
                               const DevParams& pm, int32_t* src, int32_t* type, int32_t* vid, int32_t* mult,
                               double* energy, double* grad, double* hess, hipStream_t s);

// matrix-free operator (assemble.hip): everything the two passes read
struct MfView {
    int32_t V;
    TypeRanges tr;
    const int4* st_vid;
    const int32_t* order;
    const int32_t* diag_slot;
    const int64_t* cptr;
    const uint32_t* contrib;
    const double* rec_main;
    const double* rec_extra;
    const int64_t* inc_ptr;  // per-vertex incidence offsets of the build
    const double* diag;      // per-vertex diagonal term, nullable = 0
    const double* g;         // [incidences][3] c_i w~_k, row by row (per eval)
    double2* ab;             // [Ps] (alpha, beta) of the current product (scratch)
    // dense local Hessians [Ps][12][12] (gipc_proxy_dense) instead of the
    // factors when non-null, multiplied by dense_scheme (dense.hip)
    const double* dense;
    int dense_scheme;
};
// y = (diag (x) I3 + H) x; with part, one partial of x . y per workgroup
// (mf_num_parts of them); kernels return at once when sc->done (nullable)
hipError_t launch_mf_apply(const MfView& m, const double* x, double* y, double* part, const PcgScalars* sc,
                           hipStream_t s);
hipError_t launch_mf_diag_inverse(const MfView& m, double* minv, hipStream_t s);
hipError_t launch_mf_coef(const MfView& m, double* g, hipStream_t s);
// the same product and preconditioner from m.dense (dense.hip)
hipError_t launch_dense_apply(const MfView& m, const double* x, double* y, double* part, const PcgScalars* sc,
                              hipStream_t s);
hipError_t launch_dense_diag_inverse(const MfView& m, double* minv, hipStream_t s);
int64_t mf_num_parts(int32_t V);

// dense projected proxy Hessians per staged pair, analytic or numeric
// (numeric.hip); hess [Ps][12][12]
hipError_t launch_proxy_dense(int method, const int4* st_vid, const int32_t* mult, const TypeRanges& tr,
                              const double* x, const double* xr, const DevParams& pm, double* hess, hipStream_t s);

// lagged friction (friction.hip): lag [9][Ps] at x^n; eval writes fr
// (S [Ps][8], then D and g [Ps][4]),
// grad [V][3], energy shares ev [V] and, with val, adds the blocks
hipError_t launch_fric_lag(const int4* st_vid, const int32_t* mult, const TypeRanges& tr, const double* x,
                           const double* xr, const DevParams& pm, double mu, double* lag, hipStream_t s);
hipError_t launch_fric_eval(int32_t V, const int4* st_vid, const TypeRanges& tr, const double* lag, const double* x,
                            double sv, double* fr, const int32_t* row_ptr, const int32_t* diag_slot,
                            const int64_t* cptr, const uint32_t* contrib, const int32_t* order, double* grad,
                            double* ev, void* val, int dtype, int64_t nnzb, hipStream_t s);

// contact candidates (candidates.hip)
struct CandGrid {
    double org[3];
    double h[3];
    int32_t n[3];
};
int32_t cand_bound_blocks(int64_t V, int64_t FE);
// a workgroup's part: min x y z, max x y z, largest primitive extent along
// x y z; primitives with invalid vertex ids and the first of them (triangles,
// then edges)
struct CandBounds {
    double r[9];
    int64_t nbad, first;
};
hipError_t launch_cand_bounds(const double* x, int32_t V, const int32_t* tris, int64_t F, const int32_t* edges,
                              int64_t E, CandBounds* part, int32_t nb, hipStream_t s);
// 64-byte records of the triangles and edges (box, vertex ids, object)
constexpr int kPrimRecBytes = 64;
hipError_t launch_prim_records(const double* x, const int32_t* tris, int64_t F, const int32_t* edges, int64_t E,
                               const int32_t* vobj, void* trec, void* erec, hipStream_t s);
// the cell tables of points and edges as queries (inflated by dhat), of
// triangles and of edges, one after the other: counts [4 ncell] (zero on
// entry) and the queries' numbers of cells span [V + E], then with the scanned
// counts off [4 ncell + 1] the entries ent [off[4 ncell]], a primitive
// table's in increasing id (raw [off[4 ncell] - off[2 ncell]]: scratch, fill
// [4 ncell]: zero on entry)
hipError_t launch_cells_count(const double* x, int32_t V, const int32_t* tris, int64_t F, const int32_t* edges,
                              int64_t E, const void* erec, const CandGrid& g, double dhat, int32_t* span,
                              int32_t* count, hipStream_t s);
hipError_t launch_cells_fill(const double* x, int32_t V, const int32_t* tris, int64_t F, const int32_t* edges,
                             int64_t E, const void* erec, const CandGrid& g, double dhat, const int64_t* off,
                             int32_t* fill, int32_t* raw, int32_t* ent, hipStream_t s);
// n [2 ncell]: hit-mask slots of the cells' point-triangle passes (chunks of
// 64 triangles times points), then of their edge-edge passes (chunks of 64
// queries times edges)
hipError_t launch_cell_slots(const CandGrid& g, const int64_t* off, int64_t* n, hipStream_t s);
// per cell, its queries (qtoff/qent) against its primitives (coff/cent, vertex
// ids prims, records rec): kind 0 points vs triangles, 1 edges vs edges of larger
// index; per visit e = qeoff[q] + rank of the cell in q's walk, counts into
// cnt[e] and hit masks into bal + boff[cell] (emit = false), or int32 [4]
// tuples at out + 4 eoff[e] from those masks (emit = true); evis (one per
// query-table entry) carries each visit's e from the first to the second
hipError_t launch_cell_pairs(int kind, bool emit, const double* x, const int32_t* vobj, const int32_t* prims,
                             const void* rec, const CandGrid& g, double dhat, const int64_t* qtoff,
                             const int32_t* qent, const int64_t* qeoff, const int64_t* coff, const int32_t* cent,
                             int32_t* cnt, const int64_t* eoff, const int64_t* boff, uint64_t* bal,
                             int64_t* evis, int32_t* out, hipStream_t s);

// ---- accd.hip
// additive CCD of P tuples moving by disp; counters [6] (see k_accd_reset)
hipError_t launch_accd(const int32_t* tuples, int64_t P, int32_t V, const double* x, const double* disp, double s,
                       double tc, int32_t max_iter, double* toi, unsigned long long* counters, hipStream_t st);

// ---- solve.hip
hipError_t launch_spmv(const gipc_bsr& A, const void* x, void* y, hipStream_t s);
hipError_t launch_copy(const void* src, void* dst, int64_t bytes, hipStream_t s);
// streaming read of bytes / 16 aligned 16-byte words (sink: device uint32, written only by chance)
hipError_t launch_read(const void* src, int64_t bytes, uint32_t* sink, hipStream_t s);
// with mf set, the operator is matrix-free (A is not read)
// delta = 1: stop when r.z <= rtol r0.z0 instead of ||r|| <= rtol ||b||;
// *conv (nullable) receives whether the stopping test held
hipError_t pcg_run(gipc_ctx* ctx, const gipc_bsr& A, const double* b, double* x, double rtol, int32_t maxit,
                   int32_t* iters, double* relres, int* breakdown, hipStream_t s, const MfView* mf = nullptr,
                   int delta = 0, int* conv = nullptr);
// the same on buffers carved from one device range ws of at least
// pcg_workspace_bytes(A, mf) bytes (no allocation)
size_t pcg_workspace_bytes(const gipc_bsr& A, const MfView* mf);
hipError_t pcg_run_in(void* ws, const gipc_bsr& A, const double* b, double* x, double rtol, int32_t maxit,
                      int32_t* iters, double* relres, int* breakdown, hipStream_t s, const MfView* mf = nullptr);

}  // namespace gipc
