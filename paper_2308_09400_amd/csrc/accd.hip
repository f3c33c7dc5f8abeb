// Additive CCD: the step bound of the line search (maxFeasibleStepSize in
// the implementation overview, Algorithm 1).  The paper adopts the additive
// CCD of Codimensional IPC (Li et al. 2021; Related Work, "Collision
// Detection"): a lower bound on the time of impact accumulated from safe
// sub-steps, each no longer than the current distance over a bound on how
// fast the distance can shrink.
//
// The tuple moves as x(t) = x + t p over t in [0, tc].
// With the common translation removed from p (the mean over the vertices the
// distance involves) and l_p the largest |p_i| over the first primitive plus
// the largest over the second, the distance falls at most at rate l_p.  From
// d0 = d(0) and the stop gap s d0 the lane takes a first sub-step
// (1 - s) d0 / l_p, then 0.9 d / l_p from each accepted point, until the
// distance at a trial point would fall below s d0 (the accumulated time is
// returned) or the time passes tc (tc is returned).  Distances are the
// constrained minimum of the tuple's primitives (Eq. 4 / Eq. 5), evaluated
// at each trial point from x, not accumulated.
#include <algorithm>

#include "internal.hpp"

namespace gipc {
namespace {

// 1 / v to about a unit in the last place: v_rcp_f64 and two Newton steps
__device__ __forceinline__ double recip(double v) {
    double r = __builtin_amdgcn_rcp(v);
    r = fma(fma(-v, r, 1.0), r, r);
    return fma(fma(-v, r, 1.0), r, r);
}

// squared distance of the point a + ap to the segment from a along ab, il =
// recip(l2), l2 = |ab|^2.  The parameter has to be the quotient n / l2 itself:
// one that is off by a relative 2^-45 moves the foot by 2^-45 |ab|, which is
// all of the distance where a point touches the far end (its parameter is no
// longer 1) and much of it below some 2^-40 |ab|.  So n il is corrected once by
// its remainder (Markstein's division), which gives the bits of the division
// without its scaling for the ends of the range; the products of one segment
// share the reciprocal.  On 18M tuples of sheets and of random points in all
// kinds of tuple the times have the bits that true divisions give, which cost
// 2.85 against 1.94 ms on ten 256 x 256 sheets.  A length below 7.5e-155 (its
// square has no reciprocal) counts as the first end point.
__device__ __forceinline__ double seg_near2(d3 ap, d3 ab, double l2, double il) {
    const double n = dot(ap, ab), q = n * il;
    const double a = fma(fma(-l2, q, n), il, q);
    const d3 w = ap - fmin(fmax(a, 0.0), 1.0) * ab;
    return dot(w, w);
}

// the constrained minimum of Eq. 4 / Eq. 5 over the sub-problems of
// classify_pt and classify_ee, without the sub-problem it is attained at: the
// interior tests compare numerators
__device__ __forceinline__ double near_pt2(d3 p, d3 t0, d3 t1, d3 t2) {
    const d3 e1 = t1 - t0, e2 = t2 - t0, e3 = t2 - t1, r = p - t0;
    const d3 n = cross(e1, e2);
    const double nn = dot(n, n), a11 = dot(e1, e1), a22 = dot(e2, e2), a12 = dot(e1, e2), a33 = dot(e3, e3);
    const double b1 = dot(e1, r), b2 = dot(e2, r);
    const double u = a22 * b1 - a12 * b2, v = a11 * b2 - a12 * b1, h = dot(r, n);
    double best = INFINITY;
    if (nn > kInteriorTol * a11 * a22 && u >= 0.0 && v >= 0.0 && u + v <= nn) best = h * h / nn;
    best = fmin(best, seg_near2(r, e1, a11, recip(a11)));
    best = fmin(best, seg_near2(p - t1, e3, a33, recip(a33)));
    return fmin(best, seg_near2(p - t2, t0 - t2, a22, recip(a22)));
}

__device__ __forceinline__ double near_ee2(d3 a0, d3 a1, d3 b0, d3 b1) {
    const d3 a = a1 - a0, b = b1 - b0, r = a0 - b0;
    const d3 n = cross(a, b);
    const double cc = dot(n, n), aa = dot(a, a), bb = dot(b, b);
    const double ab = dot(a, b), ar = dot(a, r), br = dot(b, r);
    const double u = ab * br - bb * ar, v = aa * br - ab * ar, h = dot(r, n);
    double best = INFINITY;
    if (cc > kInteriorTol * aa * bb && u >= 0.0 && u <= cc && v >= 0.0 && v <= cc) best = h * h / cc;
    const double ia = recip(aa), ib = recip(bb);
    best = fmin(best, seg_near2(r, b, bb, ib));
    best = fmin(best, seg_near2(a1 - b0, b, bb, ib));
    best = fmin(best, seg_near2(b0 - a0, a, aa, ia));
    return fmin(best, seg_near2(b1 - a0, a, aa, ia));
}

// constrained squared distance of a decoded tuple whose four slots are the
// local positions L[0..11] (slot k at L[3k])
__device__ __forceinline__ double local_dist2(int kind, const double* L) {
    const d3 p0 = ld3(L, 0), p1 = ld3(L, 1), p2 = ld3(L, 2), p3 = ld3(L, 3);
    if (kind == 0) return near_ee2(p0, p1, p2, p3);
    if (kind == 1) return near_pt2(p0, p1, p2, p3);
    // point against a segment (kinds 2 and 4) or a point (3 and 5)
    const bool par = kind >= 4;
    const d3 a = par ? p2 : p1, b = par ? p3 : p2;
    const d3 w = p0 - a;
    if (kind == 3 || kind == 5) return dot(w, w);
    double al;
    return seg_dist2(p0, a, b, al);
}

// counters: [0] malformed tuples, [1] first malformed index, [2] tuples
// stopped by max_iter, [3] tuples at distance 0, [4] bits of the smallest
// time (non-negative doubles order as their bit patterns), [5] largest
// number of trial steps, [6] head of the tuple queue
__global__ void k_accd_reset(unsigned long long* c, double tc) {
    if (threadIdx.x == 0) {
        c[0] = 0ull;
        c[1] = ~0ull;
        c[2] = 0ull;
        c[3] = 0ull;
        c[4] = (unsigned long long)__double_as_longlong(tc);
        c[5] = 0ull;
        c[6] = 0ull;
    }
}

// Every lane keeps one tuple's search state and takes the next tuple from a
// queue when its search has ended (a wavefront takes a chunk of queue
// entries at a time with one atomic), so a wavefront does not wait on its
// slowest lane: the searches take 1 to several hundred trial steps, and with
// one lane per tuple the ten-sheet candidates took five times as long.  A
// round of the loop forms one distance per lane, the initial one of a new
// tuple or that of a trial point, through the same code; lanes are refilled
// kAccdRefill at a time, since a round with a refill pays for its loads
// whatever their number.  A first sub-step past tc ends the search without
// its distance, which the answer does not depend on (two in five searches).
// The displacements stay in LDS, 24 registers fewer and so a fourth
// wavefront per SIMD.  Bound by vector issue (three quarters of the slots).
// The 50.6M candidates of ten 256 x 256 sheets, each falling or jittering by
// about dhat: 1.91 ms; with the initial distance apart from the trials, lanes
// refilled one at a time, a true division in every segment test and three
// atomics on one line per wavefront and 256 tuples it was 3.97 ms, and 826k
// candidates of three 101 x 101 sheets 386 against 86 us a call (there the
// atomics, 20 ns apart, were nearly all of it).
// The grid is at most the workgroups the chip holds at once; each wavefront
// starts with a chunk of its own and takes further ones from the queue until
// it is empty; every search ends within max_iter steps, so every wavefront
// does.
constexpr int kAccdRefill = 32;
constexpr int kAccdGrid = 1024;

__global__ void __launch_bounds__(kBlock, 4) k_accd_queue(const int4* __restrict__ tuples, int64_t P, int32_t V,
                                                       const double* __restrict__ X, const double* __restrict__ D,
                                                       double s, double tc, int32_t max_iter, int32_t chunk,
                                                       double* __restrict__ toi_out,
                                                       unsigned long long* __restrict__ c) {
    const int lane = threadIdx.x & 63;
    const unsigned long long below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
    // the wavefront's current chunk [cb, ce); the first ones need no atomic
    int64_t cb = ((int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6)) * chunk;
    int64_t ce = cb + chunk < P ? cb + chunk : P;
    const int64_t queue0 = (int64_t)gridDim.x * (kBlock / 64) * chunk;
    bool exhausted = false;
    bool act = false, fresh = false;  // fresh: the lane's tuple has no distance yet
    int64_t p = 0;
    int kind = 0, it = 0, itmax = 0;
    __shared__ double sdp[kBlock / 64][12][64];
    double(*dl)[64] = sdp[threadIdx.x >> 6];  // the lanes' displacements
    double x0[12];
    double lp = 0.0, g = 0.0, t = 0.0, tl = 0.0, tmin = tc;
    while (true) {
        const unsigned long long idle = __ballot(!act);
        if (!exhausted && __popcll(idle) >= kAccdRefill) {
            if (cb >= ce) {
                cb = P;
                if (queue0 < P) {
                    unsigned long long b = 0ull;
                    if (lane == 0) b = atomicAdd(&c[6], (unsigned long long)chunk);
                    cb = queue0 + (int64_t)__shfl(b, 0, 64);
                }
                ce = cb + chunk < P ? cb + chunk : P;
                exhausted = cb >= P;
            }
            const int64_t left = ce > cb ? ce - cb : 0;
            const int64_t take = (int64_t)__popcll(idle) < left ? (int64_t)__popcll(idle) : left;
            const int64_t rank = __popcll(idle & below);
            if (!act && rank < take) {
                p = cb + rank;
                int v[4], nv;
                kind = decode_tuple(tuples[p], V, v, nv);
                if (kind < 0) {
                    atomicAdd(&c[0], 1ull);
                    atomicMin(&c[1], (unsigned long long)p);
                    if (toi_out) toi_out[p] = 0.0;
                    tmin = fmin(tmin, 0.0);
                } else {
                    act = fresh = true;
                    double dp[12];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const bool use = k < nv;
                        const int vk = use ? v[k] : 0;
                        const d3 xv = ld3(X, vk), dv = ld3(D, vk);
                        x0[3 * k] = use ? xv.x : 0.0;
                        x0[3 * k + 1] = use ? xv.y : 0.0;
                        x0[3 * k + 2] = use ? xv.z : 0.0;
                        dp[3 * k] = use ? dv.x : 0.0;
                        dp[3 * k + 1] = use ? dv.y : 0.0;
                        dp[3 * k + 2] = use ? dv.z : 0.0;
                    }
                    int nf = 1, sb = 1, ns = 1;
                    switch (kind) {
                        case 0: nf = 2; sb = 2; ns = 2; break;
                        case 1: ns = 3; break;
                        case 2: ns = 2; break;
                        case 3: break;
                        case 4: sb = 2; ns = 2; break;
                        default: sb = 2; break;
                    }
                    const double im = nf + ns == 4 ? 0.25 : 0.5;  // exact
                    double m[3] = {0.0, 0.0, 0.0};
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const bool in = k < nf || (k >= sb && k < sb + ns);
#pragma unroll
                        for (int d = 0; d < 3; ++d) m[d] += in ? dp[3 * k + d] : 0.0;
                    }
#pragma unroll
                    for (int d = 0; d < 3; ++d) m[d] = nf + ns == 3 ? m[d] / 3.0 : m[d] * im;
#pragma unroll
                    for (int k = 0; k < 4; ++k)
#pragma unroll
                        for (int d = 0; d < 3; ++d) dp[3 * k + d] -= m[d];
#pragma unroll
                    for (int j = 0; j < 12; ++j) dl[j][lane] = dp[j];
                    double l1 = 0.0, l2 = 0.0;  // squared, the root taken of the largest
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const double n2 = dp[3 * k] * dp[3 * k] + dp[3 * k + 1] * dp[3 * k + 1] +
                                          dp[3 * k + 2] * dp[3 * k + 2];
                        if (k < nf) l1 = fmax(l1, n2);
                        else if (k >= sb && k < sb + ns) l2 = fmax(l2, n2);
                    }
                    lp = sqrt(l1) + sqrt(l2);
                }
            }
            cb += take;
        }
        if (__ballot(act) == 0ull) {
            if (exhausted) break;  // the queue is empty and every search has ended
            continue;
        }
        if (act) {
            const double tt = t + tl;
            const double ts = fresh ? 0.0 : tt;
            double xt[12];
#pragma unroll
            for (int j = 0; j < 12; ++j) xt[j] = fma(ts, dl[j][lane], x0[j]);
            if (fresh && !(lp > 0.0 && lp < INFINITY)) {  // a displacement that is not finite times 0 (NaN: lp = 0)
#pragma unroll
                for (int j = 0; j < 12; ++j) xt[j] = x0[j];
            }
            const double dd2 = local_dist2(kind, xt);
            bool fin = false;
            double res = 0.0;
            if (fresh) {
                fresh = false;
                if (!(dd2 > 0.0) || !(dd2 < INFINITY)) {
                    atomicAdd(&c[3], 1ull);
                    fin = true;
                } else if (lp > 0.0) {
                    const double d0 = sqrt(dd2);
                    g = s * d0;
                    t = 0.0;
                    tl = (1.0 - s) * d0 / lp;
                    it = 0;
                    if (tl > tc) {
                        res = tc;
                        fin = true;
                        itmax = max(itmax, 1);
                    }
                } else {
                    res = tc;
                    fin = true;
                }
            } else {
                ++it;
                const double dd = sqrt(dd2);
                if (t > 0.0 && dd < g) {
                    res = t;
                    fin = true;
                } else {
                    t = tt;
                    if (t > tc) {
                        res = tc;
                        fin = true;
                    } else {
                        tl = 0.9 * dd / lp;
                        if (it >= max_iter) {
                            atomicAdd(&c[2], 1ull);
                            res = t;
                            fin = true;
                        } else if (t + tl > tc && 0.1 * dd > (1.0 + 1e-9) * g) {
                            // the next trial lies past tc, and its distance,
                            // at least dd - lp tl = 0.1 dd, not below g
                            ++it;
                            res = tc;
                            fin = true;
                        }
                    }
                }
                if (fin) itmax = max(itmax, it);
            }
            if (fin) {
                if (toi_out) toi_out[p] = res;
                tmin = fmin(tmin, res);
                act = false;
            }
        }
    }
    // the workgroup's smallest time and most steps; memory only if they change it
    __shared__ double wmin[kBlock / 64];
    __shared__ int wmax[kBlock / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        tmin = fmin(tmin, __shfl_xor(tmin, o, 64));
        itmax = max(itmax, __shfl_xor(itmax, o, 64));
    }
    if (lane == 0) {
        wmin[threadIdx.x >> 6] = tmin;
        wmax[threadIdx.x >> 6] = itmax;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / 64; ++w) {
            tmin = fmin(tmin, wmin[w]);
            itmax = max(itmax, wmax[w]);
        }
        const unsigned long long tb = (unsigned long long)__double_as_longlong(tmin);
        if (tb < __hip_atomic_load(&c[4], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMin(&c[4], tb);
        if ((unsigned long long)itmax > __hip_atomic_load(&c[5], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
            atomicMax(&c[5], (unsigned long long)itmax);
    }
}

}  // namespace

hipError_t launch_accd(const int32_t* tuples, int64_t P, int32_t V, const double* x, const double* disp, double s,
                       double tc, int32_t max_iter, double* toi, unsigned long long* counters, hipStream_t st) {
    k_accd_reset<<<1, 64, 0, st>>>(counters, tc);
    if (P > 0) {
        int64_t nb = (P + kBlock - 1) / kBlock;
        if (nb > kAccdGrid) nb = kAccdGrid;
        // a quarter of a wavefront's share at once, at most 2048 tuples, so
        // that few of the queue's atomics (one line: 20 ns apart) are needed;
        // shares of up to 256 tuples are dealt out whole, without any
        const int64_t waves = nb * (kBlock / 64), share = (P + waves - 1) / waves;
        int64_t chunk = (share + 63) / 64 * 64;
        if (chunk > 256) chunk = std::min<int64_t>(2048, std::max<int64_t>(64, share / 4 / 64 * 64));
        k_accd_queue<<<(unsigned)nb, kBlock, 0, st>>>(reinterpret_cast<const int4*>(tuples), P, V, x, disp, s, tc,
                                                      max_iter, (int32_t)chunk, toi, counters);
    }
    return hipGetLastError();
}

}  // namespace gipc
