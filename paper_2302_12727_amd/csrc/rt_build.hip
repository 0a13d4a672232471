// Static geometry of the particle set: Morton order, search tree, smoothing
// lengths, wave-sliced neighbour table, particle volumes and the inverse
// least-squares matrices, global time step; point-source injection weights.
//
// Particles are static interpolation points for the radiation (Part III,
// "Using a particle based method: selecting reference frames"), so everything
// here is computed once and reused by every transport step.
#include <cstring>

#include <rocprim/rocprim.hpp>

#include <algorithm>
#include <numeric>
#include <vector>

#include "rt_internal.h"

using namespace gearrt;

namespace {

// ---------------------------------------------------------------------------
// Morton keys: 21 bits per axis, interleaved into 63 bits.
__device__ __forceinline__ uint64_t spread21(uint64_t v) {
    v &= 0x1fffffULL;
    v = (v | (v << 32)) & 0x1f00000000ffffULL;
    v = (v | (v << 16)) & 0x1f0000ff0000ffULL;
    v = (v | (v << 8)) & 0x100f00f00f00f00fULL;
    v = (v | (v << 4)) & 0x10c30c30c30c30c3ULL;
    v = (v | (v << 2)) & 0x1249249249249249ULL;
    return v;
}

__device__ __forceinline__ uint64_t morton_key(double x, double y, double z, double ibox) {
    const double v[3] = {x, y, z};
    uint64_t c[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        double f = v[a] * ibox;
        f = fmin(fmax(f, 0.0), 1.0);
        uint64_t q = (uint64_t)(f * 2097152.0);
        c[a] = q > 2097151ULL ? 2097151ULL : q;
    }
    return (spread21(c[0]) << 2) | (spread21(c[1]) << 1) | spread21(c[2]);
}

__global__ void k_morton(int64_t n, const double *__restrict__ x, double ibox,
                         uint64_t *__restrict__ keys, int32_t *__restrict__ idx) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    keys[i] = morton_key(x[3 * i], x[3 * i + 1], x[3 * i + 2], ibox);
    idx[i] = (int32_t)i;
}

__global__ void k_gather_sorted(int64_t n, const double *__restrict__ x,
                                const int32_t *__restrict__ perm, const double *__restrict__ h_in,
                                double *__restrict__ xs, double *__restrict__ h,
                                int64_t *__restrict__ perm_out) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int64_t j = perm[i];
    xs[3 * i + 0] = x[3 * j + 0];
    xs[3 * i + 1] = x[3 * j + 1];
    xs[3 * i + 2] = x[3 * j + 2];
    if (h_in) h[i] = h_in[j];
    if (perm_out) perm_out[i] = j;
}

// ---------------------------------------------------------------------------
// Search tree: leaves of kLeaf consecutive Morton-ordered particles, complete
// binary tree in heap layout above them.  Every node holds the bounding box
// of its particles and the largest compact support radius H below it.
__global__ void k_leaf_boxes(int64_t n, int64_t nleaf, int64_t P, const double *__restrict__ xs,
                             const double *__restrict__ H, double *__restrict__ lo,
                             double *__restrict__ hi, double *__restrict__ hmax) {
    int64_t l = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (l >= P) return;
    int64_t v = P + l;
    double bl[3] = {INFINITY, INFINITY, INFINITY}, bh[3] = {-INFINITY, -INFINITY, -INFINITY};
    double hm = 0.0;
    if (l < nleaf) {
        int64_t j0 = l * kLeaf, j1 = min(n, j0 + kLeaf);
        for (int64_t j = j0; j < j1; ++j) {
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                bl[a] = fmin(bl[a], xs[3 * j + a]);
                bh[a] = fmax(bh[a], xs[3 * j + a]);
            }
            if (H) hm = fmax(hm, H[j]);
        }
    }
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        lo[3 * v + a] = bl[a];
        hi[3 * v + a] = bh[a];
    }
    hmax[v] = hm;
}

__global__ void k_merge_level(int64_t first, int64_t count, double *__restrict__ lo,
                              double *__restrict__ hi, double *__restrict__ hmax) {
    int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= count) return;
    int64_t v = first + t, a = 2 * v, b = 2 * v + 1;
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        lo[3 * v + d] = fmin(lo[3 * a + d], lo[3 * b + d]);
        hi[3 * v + d] = fmax(hi[3 * a + d], hi[3 * b + d]);
    }
    hmax[v] = fmax(hmax[a], hmax[b]);
}

// Entries per particle of the neighbour lists the count pass keeps, and the
// most device memory those lists may take.
constexpr int kNList = 128;
constexpr int64_t kNListBytes = int64_t(16) << 30;
// Bits of a particle's iteration count set when its candidate list overflowed (its
// reach was cut), and when it is left to k_h_dense.
constexpr int32_t kIterOverflow = 1 << 24, kIterDense = 1 << 25;

struct Tree {
    const double *lo, *hi, *hmax;
    int64_t P;
};

// ---------------------------------------------------------------------------
// Starting point of the solve: the smaller of two density estimates (a walk
// costs about its radius cubed, so starting low is cheap and starting high is
// not):
//  - the particles per volume of the particle's leaf box (on a lattice about
//    0.7 of the root);
//  - from the fourth-nearest of the kGuessWin particles on either side in
//    Morton order, which bounds from above the distance to the fourth-nearest
//    particle, scaled by 0.8.  It stays local where a leaf straddles regions
//    of very different density and the leaf box overestimates h up to 35-fold.
constexpr int kGuessWin = 16;
__global__ void k_h_guess(int64_t n, int64_t P, const double *__restrict__ lo,
                          const double *__restrict__ hi, const double *__restrict__ xs,
                          double eta, double box, double *__restrict__ h) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    int64_t l = i / kLeaf, v = P + l;
    int64_t cnt = min((int64_t)kLeaf, n - l * kLeaf);
    double ext = 1.0;
    double floor_ext = box / 2097152.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) ext *= fmax(hi[3 * v + a] - lo[3 * v + a], floor_ext);
    double g = eta * cbrt(ext / (double)cnt);
    // four smallest r^2 in the Morton window, ascending
    const double ibox = 1.0 / box;
    const double px = xs[3 * i], py = xs[3 * i + 1], pz = xs[3 * i + 2];
    double d0 = INFINITY, d1 = INFINITY, d2 = INFINITY, d3 = INFINITY;
    const int64_t j0 = max((int64_t)0, i - kGuessWin), j1 = min(n, i + kGuessWin + 1);
    for (int64_t j = j0; j < j1; ++j) {
        if (j == i) continue;
        double sx = min_image(xs[3 * j] - px, box, ibox);
        double sy = min_image(xs[3 * j + 1] - py, box, ibox);
        double sz = min_image(xs[3 * j + 2] - pz, box, ibox);
        double r2 = sx * sx + sy * sy + sz * sz;
        if (r2 < d3) {
            d3 = r2;
            if (d3 < d2) { double t = d2; d2 = d3; d3 = t; }
            if (d2 < d1) { double t = d1; d1 = d2; d2 = t; }
            if (d1 < d0) { double t = d0; d0 = d1; d1 = t; }
        }
    }
    // n_local = 5 / ((4 pi / 3) r4^3)  ->  h = eta n_local^(-1/3)
    const double gm = eta * sqrt(d3) * 0.94269861348;      // cbrt((4 pi / 3) / 5)
    h[i] = fmin(fmin(g, 0.8 * gm), 0.25 * box);
}

// ---------------------------------------------------------------------------
// Neighbour search of one wave for up to kPts points (8 lanes each: lane =
// 8 p + c), a point p within R_p of the particles it wants (R_p < 0: none;
// HM: within max(R_p, H_j), nodes opened by their largest H).  One thread per
// particle walked a chain of some 700 dependent node and particle reads with
// every lane on lines of its own, so the search ran at the memory's latency
// (12.4 + 8.6 ms for the solve and the count of the 128^3 lattice, and 3.4 +
// 3.7 ms for 22 thousand clustered particles, which fill a third of the CUs).
// Here the wave opens the tree 6 levels at a time, one node a lane, against
// the points' bounding box; the leaves that pass are tested against each
// point (8 leaves x 8 points); the particles of the leaves left are read two
// leaves at a time, kept if they lie near the box, and collected in LDS, in
// index order, until there are 64.  emit(m) is then called with m <= 64
// candidates in B for the exact test of every point against every candidate
// (emit may shorten R, the leaves that follow are tested with that).
constexpr int kPts = 8;
template <bool HM> struct Candidates {
    double x[128], y[128], z[128], H[HM ? 128 : 1];
    int32_t j[128];
    int32_t leaf[64];
};

__device__ __forceinline__ double wave_min(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmin(v, __shfl_xor(v, o, 64));
    return v;
}
__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmax(v, __shfl_xor(v, o, 64));
    return v;
}
// Squared distance of the intervals' product [al, ah] to [bl, bh], periodic.
__device__ __forceinline__ double boxes_dist2(const double (&al)[3], const double (&ah)[3],
                                              const double *bl, const double *bh, double box) {
    double d2 = 0.0;
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const double up = bl[a] - ah[a], dn = al[a] - bh[a];   // b above a, b below a
        const double d = fmin(fmax(0.0, fmax(up, dn)),
                              fmin(fmax(0.0, up + box), fmax(0.0, dn + box)));
        d2 += d * d;
    }
    return d2;
}

template <bool HM, class Emit>
__device__ void wave_gather(const Tree &T, int depth, const double *__restrict__ xs,
                            const double *__restrict__ H, int64_t n, double box, double px,
                            double py, double pz, const double &R, Candidates<HM> &B, Emit &&emit) {
    const int lane = threadIdx.x & 63;
    const bool on = R >= 0.0;
    if (__ballot(on) == 0) return;
    const double gl[3] = {wave_min(on ? px : INFINITY), wave_min(on ? py : INFINITY),
                          wave_min(on ? pz : INFINITY)};
    const double gh[3] = {wave_max(on ? px : -INFINITY), wave_max(on ? py : -INFINITY),
                          wave_max(on ? pz : -INFINITY)};
    const double Rg = wave_max(R);
    constexpr double kSlack = 1.0 + 1e-12;      // the exact test is emit's
    int nb = 0;                                 // candidates collected
    // the accepted ones of 64 leaves v0 + lane of the tree
    auto leaves = [&](uint64_t hit, int64_t v0) {
        // hits in order, then 8 leaves x 8 points at a time
        if ((hit >> lane) & 1) B.leaf[__popcll(hit & ((uint64_t(1) << lane) - 1))] = lane;
        wave_lds_sync();
        const int nh = __popcll(hit);
        uint64_t take = 0;
        for (int t = 0; t < nh; t += 8) {
            // lane = 8 leaf + point: the point's data from lane 8 point
            const int src = 8 * (lane & 7);
            const double qx = __shfl(px, src, 64), qy = __shfl(py, src, 64),
                         qz = __shfl(pz, src, 64), qR = __shfl(R, src, 64);
            const int e = t + (lane >> 3);
            bool ok = false;
            if (e < nh && qR >= 0.0) {
                const int64_t v = v0 + B.leaf[e];
                const double rr = HM ? fmax(qR, T.hmax[v]) : qR;
                ok = box_dist2(T.lo + 3 * v, T.hi + 3 * v, qx, qy, qz, box) < rr * rr * kSlack;
            }
            const uint64_t m = __ballot(ok);
            for (int q = 0; q < 8 && t + q < nh; ++q)
                if ((m >> (8 * q)) & 0xff) take |= uint64_t(1) << (t + q);
        }
        while (take) {
            // two accepted leaves, 32 particles each
            const int e0 = __ffsll((unsigned long long)take) - 1;
            take &= take - 1;
            const int e1 = take ? __ffsll((unsigned long long)take) - 1 : -1;
            if (take) take &= take - 1;
            const int e = lane < 32 ? e0 : e1;
            bool ok = false;
            double cx = 0.0, cy = 0.0, cz = 0.0, cH = 0.0;
            int64_t j = 0;
            if (e >= 0) {
                j = (v0 + B.leaf[e] - T.P) * kLeaf + (lane & 31);
                if (j < n) {
                    cx = xs[3 * j];
                    cy = xs[3 * j + 1];
                    cz = xs[3 * j + 2];
                    double rr = Rg;
                    if (HM) {
                        cH = H[j];
                        rr = fmax(rr, cH);
                    }
                    const double c3[3] = {cx, cy, cz};
                    ok = boxes_dist2(gl, gh, c3, c3, box) < rr * rr * kSlack;
                }
            }
            const uint64_t m = __ballot(ok);
            if (ok) {
                const int pos = nb + __popcll(m & ((uint64_t(1) << lane) - 1));
                B.x[pos] = cx;
                B.y[pos] = cy;
                B.z[pos] = cz;
                if (HM) B.H[pos] = cH;
                B.j[pos] = (int32_t)j;
            }
            nb += __popcll(m);
            wave_lds_sync();
            if (nb >= 64) {
                emit(64);
                nb -= 64;
                wave_lds_sync();
                if (lane < nb) {
                    B.x[lane] = B.x[64 + lane];
                    B.y[lane] = B.y[64 + lane];
                    B.z[lane] = B.z[64 + lane];
                    if (HM) B.H[lane] = B.H[64 + lane];
                    B.j[lane] = B.j[64 + lane];
                }
                wave_lds_sync();
            }
        }
    };
    // depth first over steps of 6 levels (the first takes what is left over);
    // every node id and mask is the same in all lanes
    auto open = [&](int64_t v) {
        const double rr = HM ? fmax(Rg, T.hmax[v]) : Rg;
        return boxes_dist2(gl, gh, T.lo + 3 * v, T.hi + 3 * v, box) < rr * rr * kSlack;
    };
    const int steps = depth > 0 ? (depth + 5) / 6 : 1;
    int64_t v0[6];
    uint64_t todo[6];
    int lev = 0;
    v0[0] = int64_t(1) << (depth - 6 * (steps - 1));
    todo[0] = __ballot(lane < v0[0] && open(v0[0] + min((int64_t)lane, v0[0] - 1)));
#pragma unroll 1
    while (true) {
        if (lev == steps - 1) {
            leaves(todo[lev], v0[lev]);
            todo[lev] = 0;
        }
        while (lev >= 0 && todo[lev] == 0) --lev;
        if (lev < 0) break;
        const int c = __ffsll((unsigned long long)todo[lev]) - 1;
        todo[lev] &= todo[lev] - 1;
        const int64_t v = (v0[lev] + c) << 6;
        ++lev;
        v0[lev] = v;
        todo[lev] = __ballot(open(v + lane));
    }
    if (nb > 0) emit(nb);
}

// Sum over the 8 lanes of a point, the same bits on each of them.
__device__ __forceinline__ double sum8(double v) {
    quad_sum<4>(v);
    return v + __shfl_xor(v, 4, 64);
}

// Smoothing length: root of
//   g(h) = h^3 sum_j W(r_j, kappa h) - eta^3   (eq:number-of-neighbors),
// i.e. (sigma/kappa^3) sum_j w(r_j / (kappa h)) = eta^3, by Newton-Raphson
// safeguarded with bisection.  Iterates stay at or below hcap (compact support at
// most half the box); a root beyond it is an error.
struct HRoot {
    double pref, eta3, hcap;
    double lo = 0.0, hi = INFINITY, h;         // bracket and iterate
    __device__ HRoot(double eta, double kappa, double box, double h0)
        : pref(kSigma3 / (kappa * kappa * kappa)), eta3(eta * eta * eta),
          hcap(0.5 * box / kappa), h(fmin(h0, hcap)) {}
    // One step from the sums of w and w' q at h: true if it ends the solve (flags
    // raised on an error), else the next iterate is in hn.
    __device__ __forceinline__ bool step(double sw, double sdw, double &hn, int32_t &flags) {
        const double eps4 = 4.0 * 2.220446049250313e-16;
        const double g = pref * sw - eta3, dg = -pref * sdw / h;
        if (g == 0.0) return true;
        if (g < 0.0) lo = h; else hi = h;
        if (hi == INFINITY) {
            if (h >= hcap) {                     // g < 0 at the cap
                flags |= ST_BIGH;
                return true;
            }
            hn = 2.0 * h;                        // expand until bracketed
            if (dg > 0.0) {
                const double nt = h - g / dg;
                if (nt > h && nt < 4.0 * h) hn = nt;
            }
            hn = fmin(hn, hcap);
            return false;
        }
        // the step test comes before the bracket test: a Newton step that rounds
        // to h itself lands on a bracket end and would otherwise be replaced by a
        // bisection from a far end
        hn = dg > 0.0 ? h - g / dg : -1.0;
        if (dg > 0.0 && fabs(hn - h) <= eps4 * h) {
            h = hn;
            return true;
        }
        if (!(hn > lo && hn < hi)) hn = 0.5 * (lo + hi);
        if (fabs(hn - h) <= eps4 * h || hi - lo <= eps4 * hi) {
            h = hn;
            return true;
        }
        return false;
    }
};

// The solve of each of the wave's points from lists: the r_j < kappa h_R are
// collected once per point in LDS (kHList entries) and each sum is spread over the
// point's 8 lanes.  A point with more than kHList particles in reach cuts h_R while
// it collects and keeps the entries inside (overflow set; gathering again nearer
// in, which 45% of 22 thousand clustered particles did, took 652 us, this 248 us).
// One whose root lies beyond an h_R that was not cut gathers again further out.
// One whose root lies beyond a cut h_R does so too, cut no nearer than what is
// known to be too near, twice where a list can be expected to hold the root's
// particles (N = 4 pi (kappa eta)^3 / 3), at once where not; then it is left, with
// its iterate and dense set, to h_solve_dense.  `it` counts the evaluations before
// the last one; an evaluation at h_R that finds the root beyond it only places the
// next reach and counts neither there nor against max_iter.
constexpr int kHList = 128;
__device__ void h_solve_lists(const Tree &T, int depth, const double *__restrict__ xs, int64_t n,
                              bool on, double px, double py, double pz, double eta, double kappa,
                              double box, int32_t max_iter, Candidates<false> &B,
                              double (&list)[kPts][kHList], HRoot &r, int32_t &it, int32_t &flags,
                              bool &overflow, bool &dense) {
    const int lane = threadIdx.x & 63, p = lane >> 3, c = lane & 7;
    const double ibox = 1.0 / box;
    double hR = fmin(1.5 * r.h, r.hcap);       // the list's reach over kappa
    // short lists that were cut before a point is taken for a dense one
    int spare = 4.0 / 3.0 * kPi * kappa * kappa * kappa * r.eta3 < 0.75 * kHList ? 2 : 0;
    bool busy = on;
    dense = false;
#pragma unroll 1
    while (__ballot(busy) != 0) {
        double R = busy ? kappa * hR : -1.0, R2 = R * R;
        int cnt = 0, left = 32;                // entries; cuts of R left
        wave_gather<false>(T, depth, xs, nullptr, n, box, px, py, pz, R, B, [&](int m) {
            for (int s = 0; s < m; s += 8) {
                // no room for 8 more: the points concerned cut R (to 2/3 of the
                // volume, not below lo) and keep the entries inside; one that
                // cannot be cut to fit keeps none
                while (__ballot(cnt > kHList - 8) != 0) {
                    const bool cut = cnt > kHList - 8;
                    if (cut) {
                        overflow = true;
                        R = --left < 0 ? 0.0 : fmax(0.875 * R, 0.5 * (R + kappa * r.lo));
                        R2 = R * R;
                    }
                    int keep = 0;
                    for (int k0 = 0; k0 < kHList; k0 += 8) {
                        const double v = list[p][k0 + c];
                        const bool in = k0 + c < cnt && (!cut || v < R);
                        const uint32_t sg = (uint32_t)(__ballot(in) >> (lane & 56)) & 0xff;
                        wave_lds_sync();
                        if (in) list[p][keep + __popc(sg & ((1u << c) - 1))] = v;
                        keep += __popc(sg);
                    }
                    cnt = keep;
                    wave_lds_sync();
                }
                const int q = s + c;
                double r2 = INFINITY;
                if (q < m) {
                    const double sx = min_image(B.x[q] - px, box, ibox);
                    const double sy = min_image(B.y[q] - py, box, ibox);
                    const double sz = min_image(B.z[q] - pz, box, ibox);
                    r2 = sx * sx + sy * sy + sz * sz;
                }
                const bool hit = busy && r2 < R2;
                const uint32_t seg = (uint32_t)(__ballot(hit) >> (lane & 56)) & 0xff;
                if (hit) list[p][cnt + __popc(seg & ((1u << c) - 1))] = sqrt(r2);
                cnt += __popc(seg);
            }
        });
        wave_lds_sync();
        const bool was_cut = R < kappa * hR;
        bool probe = false;                    // h is h_R, in place of an iterate beyond it
        if (busy && was_cut) {
            hR = R / kappa;
            dense = !(hR > 0.0);               // no list fits
            busy = !dense;
            if (busy) {
                probe = r.h > hR;
                r.h = fmin(r.h, hR);
            }
        }
        // Newton-Raphson on the list, while it reaches
        bool more = busy;
        while (more) {
            if (it >= max_iter) {
                flags |= ST_NOCONV;
                busy = false;
                break;
            }
            const double iH = 1.0 / (kappa * r.h);
            double sw = 0.0, sdw = 0.0;
            for (int k = c; k < cnt; k += 8) {
                const double q = list[p][k] * iH;
                sw += kern_w(q);
                sdw += kern_dw(q) * q;
            }
            double hn;
            if (r.step(sum8(sw), sum8(sdw), hn, flags)) {
                busy = false;
                break;
            }
            if (r.hi == INFINITY && hn > hR) {
                if (r.h < hR) {
                    hn = hR;                     // the list's end first
                    probe = true;
                } else {                         // the root lies beyond
                    it -= probe;
                    hR = fmin(fmax(1.15 * hn, 1.25 * hR), r.hcap);
                    dense = was_cut && --spare < 0;
                    busy = !dense;
                    more = false;
                }
            }
            r.h = hn;
            ++it;
        }
        wave_lds_sync();
    }
}

// The solve, from the iterate r.h on, of the points with more particles at their
// root than a list holds: summed straight from the candidates of a gather per
// evaluation, none kept.  (Lists drawn out and cut again until a serial walk took
// over, 64^3 particles at eta 1.8, all of that kind, built in 54.7 ms, this way in
// 7.0; at eta 2.2 72.6 and 9.3, at eta 1.65, N = 114, 4.7 and 3.7.  Dense at the
// first short list at the default eta, N = 48: 22 thousand clustered particles
// 1.34 ms a rebuild against 1.27.)
__device__ void h_solve_dense(const Tree &T, int depth, const double *__restrict__ xs, int64_t n,
                              bool dense, double px, double py, double pz, double kappa,
                              double box, int32_t max_iter, Candidates<false> &B, HRoot &r,
                              int32_t &it, int32_t &flags) {
    const int c = threadIdx.x & 7;
    const double ibox = 1.0 / box;
#pragma unroll 1
    while (__ballot(dense) != 0) {
        if (dense && it >= max_iter) {
            flags |= ST_NOCONV;
            dense = false;
        }
        const double R = dense ? kappa * r.h : -1.0, R2 = R * R, iH = 1.0 / (kappa * r.h);
        double sw = 0.0, sdw = 0.0;
        wave_gather<false>(T, depth, xs, nullptr, n, box, px, py, pz, R, B, [&](int m) {
            for (int q = c; q < m; q += 8) {
                const double sx = min_image(B.x[q] - px, box, ibox);
                const double sy = min_image(B.y[q] - py, box, ibox);
                const double sz = min_image(B.z[q] - pz, box, ibox);
                const double r2 = sx * sx + sy * sy + sz * sz;
                if (dense && r2 < R2) {
                    const double u = sqrt(r2) * iH;
                    sw += kern_w(u);
                    sdw += kern_dw(u) * u;
                }
            }
        });
        double hn;
        sw = sum8(sw);
        sdw = sum8(sdw);
        if (dense) {
            if (r.step(sw, sdw, hn, flags)) {
                dense = false;
            } else {
                r.h = hn;
                ++it;
            }
        }
    }
}

// Smoothing lengths, one wave for 8 particles: from lists, and then the dense points
// (k_h_dense, whose waves leave at once if no point was left to it: a grid of 4
// rounds of the card's waves at most, since a wave for every 8 particles takes 56 us
// to come and go on the 128^3 lattice).  Two kernels, because a second gather in
// the first one costs it registers: 32 spilled and 2.36 ms on that lattice, against
// 2.26 without.
constexpr int64_t kDenseGrid = 4 * 256 * 12;
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_h_solve(
    int64_t n, int64_t ng, Tree T, int depth, const double *__restrict__ xs, double eta,
    double kappa, double box, double *__restrict__ h, int32_t max_iter,
    int32_t *__restrict__ iters, int32_t *__restrict__ status) {
    __shared__ Candidates<false> B;
    __shared__ double list[kPts][kHList];
    const int64_t g = xcd_block(ng);
    if (g >= ng) return;
    const int lane = threadIdx.x;
    const int64_t i = g * kPts + (lane >> 3);
    const bool on = i < n;
    const int64_t ic = on ? i : n - 1;
    int32_t it = 0, fl = 0;
    bool ovf = false, dense = false;
    HRoot r(eta, kappa, box, fmin(h[ic], 0.25 * box / kappa));
    h_solve_lists(T, depth, xs, n, on, xs[3 * ic], xs[3 * ic + 1], xs[3 * ic + 2], eta, kappa, box,
                  max_iter, B, list, r, it, fl, ovf, dense);
    if (on && (lane & 7) == 0) {
        h[i] = r.h;
        iters[i] = it | (ovf ? kIterOverflow : 0) | (dense ? kIterDense : 0);
        if (dense) fl |= ST_DENSE;
        if (fl) atomicOr(status, fl);
    }
}

__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(3, 3))) void k_h_dense(
    int64_t n, int64_t ng, Tree T, int depth, const double *__restrict__ xs, double eta,
    double kappa, double box, double *__restrict__ h, int32_t max_iter,
    int32_t *__restrict__ iters, int32_t *__restrict__ status) {
    __shared__ Candidates<false> B;
    if (!(*status & ST_DENSE)) return;
    const int lane = threadIdx.x;
    const int64_t chunk = (ng + 7) / 8;         // groups of an XCD, as xcd_block's
    for (int64_t v = blockIdx.x; v < 8 * chunk; v += gridDim.x) {
        const int64_t g = (v & 7) * chunk + (v >> 3);
        const int64_t i = g * kPts + (lane >> 3);
        const bool on = i < n;
        const int64_t ic = on ? i : n - 1;
        const int32_t word = iters[ic];
        const bool dense = on && (word & kIterDense);
        if (__ballot(dense) == 0) continue;
        int32_t it = word & (kIterOverflow - 1), fl = 0;
        HRoot r(eta, kappa, box, h[ic]);
        h_solve_dense(T, depth, xs, n, dense, xs[3 * ic], xs[3 * ic + 1], xs[3 * ic + 2], kappa,
                      box, max_iter, B, r, it, fl);
        if (dense && (lane & 7) == 0) {
            h[i] = r.h;
            iters[i] = it | kIterOverflow;
            if (fl) atomicOr(status, fl);
        }
    }
}

__global__ void k_scale(int64_t n, const double *__restrict__ a, double s, double *__restrict__ b) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) b[i] = s * a[i];
}

// ---------------------------------------------------------------------------
// Neighbour lists N(i) = { j != i : r_ij < max(H_i, H_j) }: a pair exchanges
// flux whenever one of the two kernels reaches the other particle (then
// A_ij != 0).  The count pass (one wave for 8 particles, wave_gather) keeps
// the neighbours it accepts, in index order, in a row of cap entries per
// particle: the gather neighbours (r < H_i) from its front, the others from
// its back.  The fill pass copies the rows into the table's columns and walks
// the tree itself only for the particles with more than cap neighbours.
__global__ __launch_bounds__(64) void k_neighbours_count(int64_t n, int64_t ng, Tree T, int depth,
                                                         const double *__restrict__ xs,
                                                         const double *__restrict__ H, double box,
                                                         int32_t *__restrict__ n_nbr,
                                                         int32_t *__restrict__ n_gath,
                                                         int32_t *__restrict__ list, int cap) {
    __shared__ Candidates<true> B;
    const int64_t g = xcd_block(ng);
    if (g >= ng) return;
    const int lane = threadIdx.x, c = lane & 7;
    const int64_t i = g * kPts + (lane >> 3);
    const bool on = i < n;
    const int64_t ic = on ? i : n - 1;
    const double ibox = 1.0 / box;
    const double px = xs[3 * ic], py = xs[3 * ic + 1], pz = xs[3 * ic + 2];
    const double Hi = H[ic], Hi2 = Hi * Hi;
    int32_t *row = list + ic * cap;
    int32_t cg = 0, cs = 0;
    wave_gather<true>(T, depth, xs, H, n, box, px, py, pz, on ? Hi : -1.0, B, [&](int m) {
        for (int s = 0; s < m; s += 8) {
            const int q = s + c;
            bool near = false, far = false;
            int32_t j = -1;
            if (on && q < m) {
                j = B.j[q];
                const double sx = min_image(B.x[q] - px, box, ibox);
                const double sy = min_image(B.y[q] - py, box, ibox);
                const double sz = min_image(B.z[q] - pz, box, ibox);
                const double r2 = sx * sx + sy * sy + sz * sz;
                const double Hj = B.H[q];
                near = j != (int32_t)i && r2 < Hi2;
                far = j != (int32_t)i && !near && r2 < Hj * Hj;
            }
            const uint32_t sg = (uint32_t)(__ballot(near) >> (lane & 56)) & 0xff;
            const uint32_t ss = (uint32_t)(__ballot(far) >> (lane & 56)) & 0xff;
            const int kg = cg + __popc(sg & ((1u << c) - 1));
            const int ks = cs + __popc(ss & ((1u << c) - 1));
            // (entries that would meet from both ends are not read: the fill
            // pass walks for a particle with more than cap neighbours)
            if (near && kg < cap) row[kg] = j;
            if (far && ks < cap) row[cap - 1 - ks] = j;
            cg += __popc(sg);
            cs += __popc(ss);
        }
    });
    if (on && c == 0) {
        n_nbr[i] = cg + cs;
        n_gath[i] = cg;
    }
}

__global__ void k_neighbours_fill(int64_t n, Tree T, const double *__restrict__ xs,
                                  const double *__restrict__ H, double box,
                                  const int32_t *__restrict__ n_nbr,
                                  const int32_t *__restrict__ n_gath,
                                  const int64_t *__restrict__ wave_base, int32_t *__restrict__ nbr,
                                  const int32_t *__restrict__ list, int cap) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int64_t base = wave_base[i >> 6] + (i & 63);
    const int32_t gcount = n_gath[i], scount = n_nbr[i] - gcount;
    if (gcount + scount <= cap) {
        const int32_t *row = list + i * cap;
        // full-length rows start on 16-byte boundaries
        int32_t k = 0;
        if (cap == kNList)
            for (; k + 4 <= gcount; k += 4) {
                const int4 v = *reinterpret_cast<const int4 *>(row + k);
                nbr[base + 64 * (int64_t)k] = v.x;
                nbr[base + 64 * (int64_t)(k + 1)] = v.y;
                nbr[base + 64 * (int64_t)(k + 2)] = v.z;
                nbr[base + 64 * (int64_t)(k + 3)] = v.w;
            }
        for (; k < gcount; ++k) nbr[base + 64 * (int64_t)k] = row[k];
        for (int32_t k = 0; k < scount; ++k)
            nbr[base + 64 * (int64_t)(gcount + k)] = row[cap - 1 - k];
        return;
    }
    const double ibox = 1.0 / box;
    const double px = xs[3 * i], py = xs[3 * i + 1], pz = xs[3 * i + 2];
    const double Hi = H[i], Hi2 = Hi * Hi;
    int32_t cg = 0, cs = 0;
    traverse(
        T.P,
        [&](int64_t v) {
            double R = fmax(Hi, T.hmax[v]);
            return box_dist2(T.lo + 3 * v, T.hi + 3 * v, px, py, pz, box) < R * R * (1.0 + 1e-12);
        },
        [&](int64_t l) {
            int64_t j0 = l * kLeaf, j1 = min(n, j0 + kLeaf);
            for (int64_t j = j0; j < j1; ++j) {
                if (j == i) continue;
                double sx = min_image(xs[3 * j] - px, box, ibox);
                double sy = min_image(xs[3 * j + 1] - py, box, ibox);
                double sz = min_image(xs[3 * j + 2] - pz, box, ibox);
                double r2 = sx * sx + sy * sy + sz * sz;
                double Hj = H[j];
                // the same pairs as the count pass; the bounds only keep a
                // lane inside its own column of the wave's slice
                if (r2 < Hi2) {
                    if (cg < gcount) nbr[base + 64 * (int64_t)cg] = (int32_t)j;
                    ++cg;
                } else if (r2 < Hj * Hj) {
                    if (cs < scount) nbr[base + 64 * (int64_t)(gcount + cs)] = (int32_t)j;
                    ++cs;
                }
            }
        });
}

__global__ void k_wave_width(int64_t n, int64_t nwaves, const int32_t *__restrict__ n_nbr,
                             int64_t *__restrict__ width) {
    int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (w > nwaves) return;
    if (w == nwaves) {
        width[w] = 0;
        return;
    }
    int32_t m = 0;
    int64_t i0 = w * 64, i1 = min(n, i0 + 64);
    for (int64_t i = i0; i < i1; ++i) m = max(m, n_nbr[i]);
    width[w] = 64 * (int64_t)m;
}

// ---------------------------------------------------------------------------
// Geometry (Part II "Partition of unity" and "Finite volume particle methods
// following Hopkins"): with w_ij = w(r_ij / H_i),
//   omega_i = (sigma/H_i^3) (w(0) + sum_j w_ij),  V_i = 1/omega_i,
//   E_i = sum_j s s^T psi_j(x_i) = (sigma/H_i^3) V_i S_i,  S_i = sum_j w_ij s s^T,
//   B_i = E_i^{-1} = S_i^{-1} / ((sigma/H_i^3) V_i).
// The record keeps Bv_i = V_i^2 (sigma/H_i^3) B_i = V_i S_i^{-1}, so that
//   A_kl = V_k psi~_l(x_k) - V_l psi~_k(x_l) = (w_kl Bv_k + w_lk Bv_l) s_kl.
// S_i is inverted in FP64 by cofactors.
__global__ void k_geometry(int64_t n, const double *__restrict__ xs, const double *__restrict__ h,
                           double kappa, double box, const int32_t *__restrict__ n_gath,
                           const int64_t *__restrict__ wave_base, const int32_t *__restrict__ nbr,
                           double *__restrict__ geo, float *__restrict__ geo32,
                           double *__restrict__ V_out, double *__restrict__ vol,
                           double *__restrict__ dxmin_part, int32_t *__restrict__ status) {
    __shared__ double sm[kBlock / kWave];
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    double dx = INFINITY;
    if (i < n) {
        const double ibox = 1.0 / box;
        const double px = xs[3 * i], py = xs[3 * i + 1], pz = xs[3 * i + 2];
        const double hi_ = h[i], H = kappa * hi_, iH = 1.0 / H;
        const int64_t base = wave_base[i >> 6] + (i & 63);
        const int32_t ng = n_gath[i];
        double sw = 0.0, s00 = 0, s01 = 0, s02 = 0, s11 = 0, s12 = 0, s22 = 0;
        for (int32_t k = 0; k < ng; ++k) {
            int64_t j = nbr[base + 64 * (int64_t)k];
            double sx = min_image(xs[3 * j] - px, box, ibox);
            double sy = min_image(xs[3 * j + 1] - py, box, ibox);
            double sz = min_image(xs[3 * j + 2] - pz, box, ibox);
            double r = sqrt(sx * sx + sy * sy + sz * sz);
            double w = kern_w(r * iH);
            sw += w;
            s00 += w * sx * sx; s01 += w * sx * sy; s02 += w * sx * sz;
            s11 += w * sy * sy; s12 += w * sy * sz; s22 += w * sz * sz;
        }
        double wnorm = kSigma3 * iH * iH * iH;
        double omega = wnorm * (0.5 + sw);
        double V = 1.0 / omega;
        // cofactor inverse of the symmetric S
        double c00 = s11 * s22 - s12 * s12;
        double c01 = s02 * s12 - s01 * s22;
        double c02 = s01 * s12 - s02 * s11;
        double c11 = s00 * s22 - s02 * s02;
        double c12 = s01 * s02 - s00 * s12;
        double c22 = s00 * s11 - s01 * s01;
        double det = s00 * c00 + s01 * c01 + s02 * c02;
        double tr = s00 + s11 + s22;
        if (!(det > 1e-12 * tr * tr * tr / 27.0)) {
            atomicOr(status, ST_SINGULAR);
            det = INFINITY;   // zero matrix: no gradient, no surface from this side
        }
        double f = V / det;
        double *rec = geo + (int64_t)kRec * i;
        rec[R_X + 0] = px;
        rec[R_X + 1] = py;
        rec[R_X + 2] = pz;
        rec[R_IH] = iH;
        rec[R_H] = hi_;
        rec[R_V] = V;
        rec[R_B + 0] = f * c00;
        rec[R_B + 1] = f * c01;
        rec[R_B + 2] = f * c02;
        rec[R_B + 3] = f * c11;
        rec[R_B + 4] = f * c12;
        rec[R_B + 5] = f * c22;
        rec[12] = rec[13] = rec[14] = rec[15] = 0.0;
        if (geo32) {
            float *r32 = geo32 + (int64_t)F_REC * i;
            double *xd = reinterpret_cast<double *>(r32);
            xd[0] = px;
            xd[1] = py;
            xd[2] = pz;
            r32[F_IH] = (float)iH;
            r32[F_H] = (float)hi_;
            r32[F_B + 0] = (float)(f * c00);
            r32[F_B + 1] = (float)(f * c01);
            r32[F_B + 2] = (float)(f * c02);
            r32[F_B + 3] = (float)(f * c11);
            r32[F_B + 4] = (float)(f * c12);
            r32[F_B + 5] = (float)(f * c22);
            r32[F_V] = (float)V;
            r32[15] = 0.0f;
        }
        V_out[i] = V;
        vol[i] = V;   // compact copy for the per-particle kernels that need nothing else
        dx = cbrt(V * (3.0 / (4.0 * kPi)));
    }
    // block minimum of dx
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) dx = fmin(dx, __shfl_down(dx, o, 64));
    if ((threadIdx.x & 63) == 0) sm[threadIdx.x >> 6] = dx;
    __syncthreads();
    if (threadIdx.x == 0) {
        double m = sm[0];
        for (int w = 1; w < kBlock / kWave; ++w) m = fmin(m, sm[w]);
        dxmin_part[blockIdx.x] = m;
    }
}

__global__ void k_dt(int64_t nb, const double *__restrict__ part, double cfl, double c,
                     double *__restrict__ dt) {
    __shared__ double sm[kBlock];
    double m = INFINITY;
    for (int64_t b = threadIdx.x; b < nb; b += blockDim.x) m = fmin(m, part[b]);
    sm[threadIdx.x] = m;
    __syncthreads();
    for (int s = blockDim.x / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) sm[threadIdx.x] = fmin(sm[threadIdx.x], sm[threadIdx.x + s]);
        __syncthreads();
    }
    if (threadIdx.x == 0) dt[0] = cfl * sm[0] / c;
}

__global__ void k_copy_dt(const double *__restrict__ a, double *__restrict__ b) { b[0] = a[0]; }

// ---------------------------------------------------------------------------
// Sources (Part III "Weights for distribution of energy density of a star onto
// particles"): smoothing length of the source over the gas, then
//   psi_sg = W(r_sg, H_s) / sum_g' W(r_sg', H_s),
//   octant a(g) from the signs of x_g - x_s (components >= 0 count as +),
//   w_a = sum_{g in a} psi_sg,  mu_a = sum_b w_b / (q_nz w_a),
//   xi_sg = mu_a psi_sg   (eq:isotropy-correction-with-zero).
// One wave per source (h of the gas particle nearest in Morton order as the
// start): with one thread per source the walks' latency made this the longest
// kernel of a clustered build (11.3 ms for 64 sources among 58 thousand
// particles).
__global__ __launch_bounds__(64) void k_src_h(int32_t S, Tree T, int depth,
                                              const double *__restrict__ xs, int64_t n,
                                              const uint64_t *__restrict__ keys,
                                              const double *__restrict__ geo,
                                              const double *__restrict__ src_x, double eta,
                                              double kappa, double box, int32_t max_iter,
                                              double *__restrict__ src_h,
                                              int32_t *__restrict__ status) {
    __shared__ Candidates<false> B;
    __shared__ double list[kPts][kHList];
    const int32_t s = blockIdx.x;
    const double px = src_x[3 * s], py = src_x[3 * s + 1], pz = src_x[3 * s + 2];
    const uint64_t key = morton_key(px, py, pz, 1.0 / box);
    int64_t lo = 0, hi = n - 1;                 // first particle with keys[i] >= key
    while (lo < hi) {
        const int64_t m = (lo + hi) >> 1;
        if (keys[m] < key) lo = m + 1;
        else hi = m;
    }
    int32_t it = 0, fl = 0;
    bool ovf = false, dense = false;
    HRoot r(eta, kappa, box, fmin(geo[(int64_t)kRec * lo + R_H], 0.25 * box / kappa));
    h_solve_lists(T, depth, xs, n, threadIdx.x < 8, px, py, pz, eta, kappa, box, max_iter, B, list,
                  r, it, fl, ovf, dense);
    h_solve_dense(T, depth, xs, n, dense, px, py, pz, kappa, box, max_iter, B, r, it, fl);
    if (threadIdx.x == 0) {
        src_h[s] = r.h;
        if (fl) atomicOr(status, fl);
    }
}

// Gas particles within H_s of each source (cnt), or with FILL their indices,
// injection weights xi and coefficients xi / V; one wave per source.
template <bool FILL>
__global__ __launch_bounds__(64) void k_src_gas(int32_t S, Tree T, int depth,
                                                const double *__restrict__ xs, int64_t n,
                                                const double *__restrict__ src_x,
                                                const double *__restrict__ src_h, double kappa,
                                                double box, const double *__restrict__ geo,
                                                int32_t *__restrict__ cnt,
                                                const int32_t *__restrict__ ptr,
                                                int32_t *__restrict__ gas, double *__restrict__ xi,
                                                double *__restrict__ coef) {
    __shared__ Candidates<false> B;
    const int32_t s = blockIdx.x;
    const int lane = threadIdx.x;
    const double ibox = 1.0 / box;
    const double px = src_x[3 * s], py = src_x[3 * s + 1], pz = src_x[3 * s + 2];
    const double H = kappa * src_h[s], H2 = H * H, iH = 1.0 / H;
    int32_t c = 0;
    const int32_t o = FILL ? ptr[s] : 0;
    const int32_t cap = FILL ? ptr[s + 1] - ptr[s] : 0;
    double wa[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    wave_gather<false>(T, depth, xs, nullptr, n, box, px, py, pz, lane < 8 ? H : -1.0, B,
                       [&](int m) {
        // a candidate a lane
        bool hit = false;
        double sx = 0.0, sy = 0.0, sz = 0.0, r2 = 0.0;
        if (lane < m) {
            sx = min_image(B.x[lane] - px, box, ibox);
            sy = min_image(B.y[lane] - py, box, ibox);
            sz = min_image(B.z[lane] - pz, box, ibox);
            r2 = sx * sx + sy * sy + sz * sz;
            hit = r2 < H2;
        }
        const uint64_t hits = __ballot(hit);
        if (FILL && hit) {
            const int32_t e = c + __popcll(hits & ((uint64_t(1) << lane) - 1));
            if (e < cap) {
                const double w = kern_w(sqrt(r2) * iH);
                const int oc = (sx >= 0.0) | ((sy >= 0.0) << 1) | ((sz >= 0.0) << 2);
                gas[o + e] = B.j[lane];
                xi[o + e] = w;
                coef[o + e] = (double)oc;   // octant, replaced below
#pragma unroll
                for (int a = 0; a < 8; ++a) wa[a] += a == oc ? w : 0.0;
            }
        }
        c += __popcll(hits);
    });
    if (!FILL) {
        if (lane == 0) cnt[s] = c;
        return;
    }
    int qnz = 0;
#pragma unroll
    for (int a = 0; a < 8; ++a) {
#pragma unroll
        for (int d = 32; d > 0; d >>= 1) wa[a] += __shfl_xor(wa[a], d, 64);
        qnz += wa[a] > 0.0;
    }
    // xi_sg = mu_a psi_sg with psi_sg = w_sg / wsum and w_a in units of wsum:
    // mu_a psi_sg = (wsum / (q_nz wa_a)) (w_sg / wsum) = w_sg / (q_nz wa_a)
    if (c > cap) c = cap;
    __syncthreads();                            // the entries are other lanes' writes
    for (int32_t e = lane; e < c; e += 64) {
        const int oc = (int)coef[o + e];
        double wo = 0.0;
#pragma unroll
        for (int a = 0; a < 8; ++a) wo = a == oc ? wa[a] : wo;
        const double x_ = xi[o + e] > 0.0 ? xi[o + e] / ((double)qnz * wo) : 0.0;
        xi[o + e] = x_;
        coef[o + e] = x_ / geo[(int64_t)kRec * gas[o + e] + R_V];
    }
}

// The value of lane l (the same l in every lane), and of a 64-bit one.
__device__ __forceinline__ int32_t lane_value(int32_t v, int l) {
    return __builtin_amdgcn_readlane(v, l);
}
__device__ __forceinline__ uint64_t lane_value64(uint64_t v, int l) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, l);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), l);
    return ((uint64_t)hi << 32) | lo;
}

// Second pass of the task lists: lower the tile's longest list, which sets
// how long the tile's block runs, by augmenting paths.  A particle k with the
// longest list (L entries) passes one of the pairs it evaluates, (k, l), to l;
// if l's list is not at least 2 shorter than L, l passes one of its own on,
// and so on along a breadth-first path (lowest indices first) that ends at a
// particle with at most L - 2 entries: k's list shrinks by one, the end's
// grows by one, the others keep their length.  Repeated while some particle
// with the longest list has such a path; each move lowers the sum of the
// squared lengths, so the loop ends.  On the lattices this reaches the lower
// bound, the larger of the longest list of neighbours outside the tile and
// the mean, in all but a few tiles.  One wave (lane = particle of the tile);
// c: the lane's list length, bit l of own: the lane evaluates its pair with l,
// adj: the lane's partners in the tile.  All in registers: u evaluates the
// pair (u, lane) when adj has u and own has not, so a lane finds the particles
// of the frontier that can pass it a pair with two bit operations.
__device__ __forceinline__ void level_tasks(bool active, int lane, int32_t &c, uint64_t &own,
                                            uint64_t adj) {
    for (int guard = 0; guard < 64 * 64; ++guard) {
        int32_t top = active ? c : -1;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) top = max(top, __shfl_xor(top, o, 64));
        uint64_t tops = __ballot(active && c == top);
        bool moved = false;
        while (tops && !moved) {
            const int v = __ffsll((unsigned long long)tops) - 1;
            tops &= tops - 1;
            uint64_t visited = uint64_t(1) << v, frontier = visited;
            int found = -1;
            int32_t prev = -1;                  // the lane that can pass this one a pair
            while (frontier && found < 0) {
                const uint64_t from = adj & ~own & frontier;
                const bool reach = from != 0 && !((visited >> lane) & 1);
                if (reach) prev = __ffsll((unsigned long long)from) - 1;
                const uint64_t disc = __ballot(reach);
                const uint64_t good = __ballot(reach && c <= top - 2);
                if (good) found = __ffsll((unsigned long long)good) - 1;
                visited |= disc;
                frontier = disc;
            }
            if (found >= 0) {
                for (int w = found; w != v;) {
                    const int u = lane_value(prev, w);
                    if (lane == u) own &= ~(uint64_t(1) << w);
                    if (lane == w) own |= uint64_t(1) << u;
                    w = u;
                }
                c += (lane == found) - (lane == v);
                moved = true;
            }
        }
        if (!moved) break;
    }
}

// Task lists of the tile transport (k_transport64_tile): particle i's
// neighbours outside its tile (kTile consecutive particles within its
// 64-particle column block of the neighbour table) and, flagged by the sign
// bit, the tile partners it evaluates for both.  Which of the two evaluates
// an in-tile pair is chosen to balance the lists, whose longest in each
// group of 16 particles (one wave of the transport, 8 at 8 lanes a particle)
// sets the iterations of a pass: one wave per tile starts from each particle's count
// of neighbours outside the tile and gives the tile's pairs, in a fixed order
// (by the lower index, then by its list order), one by one to the particle
// with the shorter list so far (the lower index on ties); level_tasks then
// lowers the tile's longest list.  On the 32^3 lattice the greedy pass takes
// the mean wave iterations of the transport to 0.75 of the two-sided
// kernel's (a fixed rule by index parity took them to 0.82 on the 64^3
// lattice) and the longest list of a tile, which sets its block's time, to
// 0.81; the leveling takes them to 0.70 and 0.69.  Same slots as the neighbour
// table, in table order; n_task[i] entries.  Launched with one wave (64
// threads) per tile.  The tile's pairs are kept as bit masks in registers and
// handed out with scalar lane reads: with the lists read by one lane at a time
// and the counts in LDS this was a serial chain of LDS and memory reads, 5.5 ms
// on the 128^3 lattice and 0.51 ms on 22 thousand clustered particles; now 1.21
// and 0.13 ms, with the same lists.
__global__ __launch_bounds__(64) void k_tasks(int64_t n, const int64_t *__restrict__ wave_base,
                                              const int32_t *__restrict__ n_nbr,
                                              const int32_t *__restrict__ n_gath,
                                              const int32_t *__restrict__ nbr,
                                              int32_t *__restrict__ task,
                                              int32_t *__restrict__ n_task,
                                              int64_t *__restrict__ tstat) {
    static_assert(kTile == 64, "a tile is one column block of the neighbour table");
    const int lane = threadIdx.x;
    const int64_t t0 = (int64_t)blockIdx.x * 64, i = t0 + lane;
    const bool active = i < n;
    const int64_t base = wave_base[blockIdx.x] + lane;
    const int32_t nn = active ? n_nbr[i] : 0, ng = active ? n_gath[i] : 0;
    uint64_t adjg = 0, adjs = 0;                // partners in the tile: gather ones, others
    for (int32_t k = 0; k < nn; ++k) {
        const int32_t jl = nbr[base + 64 * (int64_t)k] - (int32_t)t0;
        const uint64_t bit = (uint32_t)jl < 64u ? uint64_t(1) << (jl & 63) : 0;
        if (k < ng) adjg |= bit;
        else adjs |= bit;
    }
    const uint64_t adj = adjg | adjs;
    const int32_t out = nn - __popcll(adj);
    int32_t c = out;
    uint64_t own = 0;                           // bit l: this particle evaluates its pair with l
    for (int src = 0; src < 63; ++src) {
        int32_t ci = lane_value(c, src);
        uint64_t mine = 0;
        const uint64_t above = ~uint64_t(0) << (src + 1);
#pragma unroll
        for (int part = 0; part < 2; ++part)
            for (uint64_t m = lane_value64(part ? adjs : adjg, src) & above; m; m &= m - 1) {
                const int l = __ffsll((unsigned long long)m) - 1;
                if (lane_value(c, l) < ci) {
                    if (lane == l) {
                        ++c;
                        own |= uint64_t(1) << src;
                    }
                } else {
                    ++ci;
                    mine |= uint64_t(1) << l;
                }
            }
        if (lane == src) {
            c = ci;
            own |= mine;
        }
    }
    level_tasks(active, lane, c, own, adj);
    {
        // the tile's longest list and its lower bound: the longest list of
        // neighbours outside the tile, or the mean length rounded up
        int32_t lm = active ? c : 0, om = out, sm = lm, na = active ? 1 : 0;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) {
            lm = max(lm, __shfl_xor(lm, o, 64));
            om = max(om, __shfl_xor(om, o, 64));
            sm += __shfl_xor(sm, o, 64);
            na += __shfl_xor(na, o, 64);
        }
        if (lane == 0 && na > 0) {
            atomicAdd((unsigned long long *)&tstat[0], (unsigned long long)lm);
            atomicAdd((unsigned long long *)&tstat[1],
                      (unsigned long long)max(om, (sm + na - 1) / na));
        }
    }
    if (!active) return;
    int32_t o = 0;
    for (int32_t k = 0; k < nn; ++k) {
        int32_t j = nbr[base + 64 * (int64_t)k];
        const int32_t jl = j - (int32_t)t0;
        if ((uint32_t)jl < 64u) {
            if (!((own >> jl) & 1)) continue;
            j |= int32_t(0x80000000u);
        }
        task[base + 64 * (int64_t)o] = j;
        ++o;
    }
    n_task[i] = o;
}

// Neighbour unions of the gradient (k_gradient64u, k_gradient32u; over the
// gather lists) and of the adjoint's transposed gradient (k_adj_grad64u; over
// the symmetric lists): for every block of 64 particles (a column block of the
// neighbour table) the sorted distinct indices of its particles and of the
// first len[i] neighbours of each, which the kernel stages in LDS once instead
// of fetching a neighbour's row for every pair (each row is used 6-8 times by
// a block).  Each of those slots gets the 16-bit position of its neighbour in
// the union (gloc, packed, see rt_ctx), each particle its own (uown).  Block b's
// rows go to urow[b cap ..], rows[b] of them, 0 if there are more than cap (the
// block is left to the staged kernel).  The distinct indices are collected in
// an LDS hash table (open addressing) and sorted (bitonic);
// a key's position is kept beside it in the table, where its slots find it.
// One block of 256 threads (4 per particle) per 64-particle block.  (A count
// pass, a sort of 1024 keys whatever their number and a binary search per slot
// took 2.6 ms for both unions of the 128^3 lattice, this 1.2 ms.)  blist: only
// the listed blocks, whose rows go to urow and rows in the order of the list.
constexpr int kUnionHash = 2048;

__global__ __launch_bounds__(256) void k_union(int64_t n, int64_t nb, int cap,
                                               const int64_t *__restrict__ wave_base,
                                               const int32_t *__restrict__ len,
                                               const int32_t *__restrict__ nbr,
                                               int32_t *__restrict__ rows,
                                               int32_t *__restrict__ urow,
                                               const int64_t *__restrict__ goff,
                                               uint16_t *__restrict__ gloc,
                                               uint16_t *__restrict__ uown,
                                               const int32_t *__restrict__ blist = nullptr) {
    __shared__ int32_t keys[kUnionHash];
    __shared__ uint16_t val[kUnionHash];
    __shared__ int32_t srt[kUnionSort];
    __shared__ int32_t cnt;
    const int64_t bx = xcd_block(nb);
    if (bx >= nb) return;                       // whole block
    const int64_t b = blist ? (int64_t)blist[bx] : bx, t0 = b * 64;
    for (int e = threadIdx.x; e < kUnionHash; e += 256) keys[e] = -1;
    if (threadIdx.x == 0) cnt = 0;
    __syncthreads();
    const int p = threadIdx.x >> 2, sub = threadIdx.x & 3;
    const int64_t i = t0 + p;
    const bool active = i < n;
    const int64_t base = wave_base[b] + p;
    const int32_t ng = active ? len[i] : 0;
    auto slot_of = [](int32_t j) { return ((uint32_t)j * 2654435761u) >> 21; };   // 11 bits
    auto insert = [&](int32_t j) {
        uint32_t h = slot_of(j);
        // (with more than cap keys the block is given up, so the table, at
        // least half of which is free until then, cannot fill before)
        while (*(volatile int32_t *)&cnt <= cap) {
            // (most are there already: a read is cheaper than the exchange)
            int32_t old = *(volatile int32_t *)&keys[h];
            if (old == -1) old = atomicCAS(&keys[h], -1, j);
            if (old == -1) {
                // (a slot's first key: listed in any order, sorted next)
                const int32_t pos = atomicAdd(&cnt, 1);
                if (pos < kUnionSort) srt[pos] = j;
                return;
            }
            if (old == j) return;
            h = (h + 1) & (kUnionHash - 1);
        }
    };
    if (active && sub == 0) insert((int32_t)i);
    for (int32_t k = sub; k < ng; k += 4) insert(nbr[base + 64 * (int64_t)k]);
    __syncthreads();
    const int32_t m = cnt;
    const bool fits = m <= cap;                             // block-uniform
    if (threadIdx.x == 0) rows[bx] = fits ? m : 0;
    if (!fits) return;
    int size = 64;
    while (size < m) size <<= 1;
    for (int e = m + threadIdx.x; e < size; e += 256) srt[e] = INT32_MAX;
    __syncthreads();
    for (int k = 2; k <= size; k <<= 1)
        for (int jj = k >> 1; jj > 0; jj >>= 1) {
            for (int e = threadIdx.x; e < size; e += 256) {
                const int l = e ^ jj;
                if (l > e) {
                    const int32_t u = srt[e], c = srt[l];
                    if ((u > c) == ((e & k) == 0)) {
                        srt[e] = c;
                        srt[l] = u;
                    }
                }
            }
            __syncthreads();
        }
    auto find = [&](int32_t j) {                            // j is in the table
        uint32_t h = slot_of(j);
        while (keys[h] != j) h = (h + 1) & (kUnionHash - 1);
        return h;
    };
    for (int e = threadIdx.x; e < m; e += 256) {
        const int32_t j = srt[e];
        urow[bx * cap + e] = j;
        val[find(j)] = (uint16_t)e;
    }
    __syncthreads();
    if (active && sub == 0) uown[i] = val[find((int32_t)i)];
    // 4 slots of a lane are one 8-byte store (those past its last are not read)
    uint16_t *g = gloc + goff[b] + 4 * (int64_t)threadIdx.x;   // lane 4p + sub
    for (int32_t k = sub; k < ng; k += 16) {
        uint64_t v = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            if (k + 4 * q < ng)
                v |= (uint64_t)val[find(nbr[base + 64 * (int64_t)(k + 4 * q)])] << (16 * q);
        *reinterpret_cast<uint64_t *>(g + (int64_t)(k >> 4) * 1024) = v;
    }
}

// Packed table entries of every block (goff[b + 1] - goff[b]): 1024 per group
// of 16 table rows.
__global__ void k_union_width(int64_t nw, const int64_t *__restrict__ wave_base,
                              int64_t *__restrict__ width) {
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b > nw) return;
    width[b] = b == nw ? 0 : 1024 * (((wave_base[b + 1] - wave_base[b]) / 64 + 15) / 16);
}

// The blocks with more than cap rows or none (left to the staged kernel), in
// order, with cap = cap3 (three waves per SIMD) if at least 95% of the blocks
// fit it: out[0] how many, out[1] the waves per SIMD, then the list (ids: of the
// blocks so named).  One block.
__global__ __launch_bounds__(1024) void k_union_left(int64_t nw, const int32_t *__restrict__ rows,
                                                     int w0, int cap3, int32_t *__restrict__ out,
                                                     const int32_t *__restrict__ ids = nullptr) {
    __shared__ int32_t sm[1024];
    __shared__ int32_t base;
    const int t = threadIdx.x;
    int32_t fit = 0;
    for (int64_t b = t; b < nw; b += 1024) fit += rows[b] > 0 && rows[b] <= cap3;
    sm[t] = fit;
    __syncthreads();
    for (int o = 512; o > 0; o >>= 1) {
        if (t < o) sm[t] += sm[t + o];
        __syncthreads();
    }
    const bool three = cap3 > 0 && sm[0] >= nw - nw / 20;
    if (t == 0) base = 0;
    __syncthreads();
    for (int64_t b0 = 0; b0 < nw; b0 += 1024) {
        const int64_t b = b0 + t;
        const int32_t r = b < nw ? rows[b] : 1;
        const bool left = b < nw && (r == 0 || (three && r > cap3));
        const uint64_t m = __ballot(left);
        const int wv = t >> 6, lane = t & 63;
        if (lane == 0) sm[wv] = __popcll(m);
        __syncthreads();
        int32_t at = base;
        for (int w = 0; w < wv; ++w) at += sm[w];
        if (left) out[2 + at + __popcll(m & ((uint64_t(1) << lane) - 1))] =
                      ids ? ids[b] : (int32_t)b;
        __syncthreads();
        if (t == 0)
            for (int w = 0; w < 16; ++w) base += sm[w];
        __syncthreads();
    }
    if (t == 0) {
        out[0] = base;
        out[1] = three ? 3 : w0;
    }
}

// Statistics of a build, one block's share added to s: neighbour entries,
// gather entries, particles whose candidate list overflowed; the most
// neighbours of a particle and the most iterations in mx.
__global__ __launch_bounds__(kBlock) void k_stats(int64_t n, const int32_t *__restrict__ n_nbr,
                                                  const int32_t *__restrict__ n_gath,
                                                  const int32_t *__restrict__ iters,
                                                  BuildResult *__restrict__ r) {
    int64_t a = 0, g = 0, o = 0;
    int32_t mn = 0, mi = 0;
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n; i += (int64_t)gridDim.x * kBlock) {
        const int32_t k = n_nbr[i], it = iters[i];
        a += k;
        g += n_gath[i];
        o += (it & kIterOverflow) != 0;
        mn = max(mn, k);
        mi = max(mi, it & (kIterOverflow - 1));
    }
    a = wave_sum_i64(a);
    g = wave_sum_i64(g);
    o = wave_sum_i64(o);
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        mn = max(mn, __shfl_down(mn, d, 64));
        mi = max(mi, __shfl_down(mi, d, 64));
    }
    // one atomic per block and number: they all go to one line
    __shared__ int64_t part[kBlock / 64][5];
    const int wv = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) {
        part[wv][0] = a;
        part[wv][1] = g;
        part[wv][2] = o;
        part[wv][3] = mn;
        part[wv][4] = mi;
    }
    __syncthreads();
    const int k = threadIdx.x;
    if (k < 5) {
        unsigned long long v = 0;
        for (int w = 0; w < kBlock / 64; ++w) {
            const unsigned long long u = (unsigned long long)part[w][k];
            v = k < 3 ? v + u : max(v, u);
        }
        if (k < 3) atomicAdd(&r->stat[k], v);
        else atomicMax(&r->stat[k], v);
    }
}

// The rest of what the host reads once a build is done.
__global__ void k_result(const int32_t *__restrict__ status, const int32_t *__restrict__ left,
                         const int32_t *__restrict__ aleft, BuildResult *__restrict__ r) {
    r->status = *status;
    for (int k = 0; k < 2; ++k) {
        r->left[k] = left ? left[k] : 0;
        r->aleft[k] = aleft ? aleft[k] : 0;
    }
}

inline unsigned nblk(int64_t n, int b = kBlock) { return (unsigned)((n + b - 1) / b); }

}  // namespace

// ---------------------------------------------------------------------------
// host side

static int tree_depth(const rt_ctx *ctx) {
    int d = 0;
    while ((int64_t(1) << d) < ctx->P) ++d;
    return d;
}

static void build_tree(rt_ctx *ctx, const double *H) {
    int64_t P = ctx->P;
    k_leaf_boxes<<<nblk(P), kBlock, 0, ctx->stream>>>(ctx->p.n, ctx->nleaf, P, ctx->xs, H,
                                                      ctx->node_lo, ctx->node_hi, ctx->node_hmax);
    for (int64_t first = P / 2; first >= 1; first /= 2)
        k_merge_level<<<nblk(first), kBlock, 0, ctx->stream>>>(first, first, ctx->node_lo,
                                                               ctx->node_hi, ctx->node_hmax);
}

rt_status rt_build_impl(rt_ctx *ctx, const double *x, const double *h_in, int64_t *perm,
                        double *h, double *V, double *dt) {
    const int64_t n = ctx->p.n;
    hipStream_t st = ctx->stream;
    rt_status rs;
    ctx->built = 0;
    ctx->nleaf = (n + kLeaf - 1) / kLeaf;
    ctx->P = 1;
    while (ctx->P < ctx->nleaf) ctx->P *= 2;
    const int64_t nw = ctx->nwaves = (n + 63) / 64;
    const bool f64 = ctx->p.precision == RT_FP64;
    const int G = ctx->p.groups;
    const int ucap = f64 ? union_cap(G) : union_cap32(G), ucap3 = f64 ? union_cap3(G) : 0;
    const int acap = f64 && ucap > 0 ? adj_union_cap(2) : 0;

    // The context's arrays outlive the build and serve the next one (a moved
    // particle set has as many particles).  What the sort, the searches and the
    // scans need lies in the geometry records, which are written last, and the
    // statistics are summed on the device: with arrays allocated anew, counts
    // copied back and summed and union offsets made by the host, a rebuild of
    // the 128^3 lattice and a step took 31.6 ms, this 12.4 ms.
    char *list_mem = nullptr;
    size_t sort_bytes = 0, scan_bytes = 0;
    BuildResult res{};
    // (no work queued on a stream the context had before reads what this build
    // writes)
    if (ctx->xs) RT_HIP(hipDeviceSynchronize());

#define RESERVE(p, bytes)                                                  \
    do {                                                                   \
        if ((rs = rt_reserve(ctx, (void **)&(p), (bytes))) != RT_OK) goto fail; \
    } while (0)
#define HIP_OR_FAIL(expr)                                                  \
    do {                                                                   \
        const hipError_t e_ = (expr);                                      \
        if (e_ != hipSuccess) {                                            \
            rs = rt_fail(ctx, RT_EHIP, std::string(#expr) + ": " + hipGetErrorString(e_)); \
            goto fail;                                                     \
        }                                                                  \
    } while (0)

    RESERVE(ctx->xs, sizeof(double) * 3 * n);
    if (!f64) RESERVE(ctx->geo32, sizeof(float) * F_REC * n);
    RESERVE(ctx->vol, sizeof(double) * n);
    RESERVE(ctx->perm32, sizeof(int32_t) * n);
    RESERVE(ctx->keys, sizeof(uint64_t) * n);
    RESERVE(ctx->h_iters, sizeof(int32_t) * n);
    RESERVE(ctx->node_lo, sizeof(double) * 3 * 2 * ctx->P);
    RESERVE(ctx->node_hi, sizeof(double) * 3 * 2 * ctx->P);
    RESERVE(ctx->node_hmax, sizeof(double) * 2 * ctx->P);
    RESERVE(ctx->n_nbr, sizeof(int32_t) * n);
    RESERVE(ctx->n_gath, sizeof(int32_t) * n);
    RESERVE(ctx->wave_base, sizeof(int64_t) * (nw + 1));
    RESERVE(ctx->n_task, sizeof(int32_t) * n);
    RESERVE(ctx->tstat, 2 * sizeof(int64_t));
    RESERVE(ctx->dxpart, sizeof(double) * nblk(n));
    RESERVE(ctx->result, sizeof(BuildResult));
    if (ucap > 0) {
        RESERVE(ctx->goff, sizeof(int64_t) * (nw + 1));
        RESERVE(ctx->urows, sizeof(int32_t) * nw);
        RESERVE(ctx->urow, sizeof(int32_t) * nw * ucap);
        RESERVE(ctx->uown, sizeof(uint16_t) * n);
        RESERVE(ctx->ublk, sizeof(int32_t) * (nw + 2));
    }
    if (acap > 0) {
        RESERVE(ctx->arows, sizeof(int32_t) * nw);
        RESERVE(ctx->arow, sizeof(int32_t) * nw * acap);
        RESERVE(ctx->aown, sizeof(uint16_t) * n);
        RESERVE(ctx->ablk, sizeof(int32_t) * (nw + 2));
    }
    {
        // 256-byte aligned pieces
        if (rocprim::radix_sort_pairs(nullptr, sort_bytes, (uint64_t *)nullptr, (uint64_t *)nullptr,
                                      (int32_t *)nullptr, (int32_t *)nullptr, (size_t)n, 0, 63,
                                      st) != hipSuccess ||
            rocprim::exclusive_scan(nullptr, scan_bytes, (int64_t *)nullptr, (int64_t *)nullptr,
                                    (int64_t)0, (size_t)(nw + 1), rocprim::plus<int64_t>(),
                                    st) != hipSuccess) {
            rs = rt_fail(ctx, RT_EHIP, "sort or scan size query failed");
            goto fail;
        }
        size_t total = 0;
        auto piece = [&](size_t bytes) {
            const size_t at = total;
            total += (bytes + 255) / 256 * 256;
            return at;
        };
        const size_t at_keys = piece(sizeof(uint64_t) * n), at_idx = piece(sizeof(int32_t) * n),
                     at_H = piece(sizeof(double) * n), at_width = piece(sizeof(int64_t) * (nw + 1)),
                     at_work = piece(std::max(sort_bytes, scan_bytes));
        RESERVE(ctx->geo, std::max(total, sizeof(double) * kRec * n));
        char *tmp = (char *)ctx->geo;
        uint64_t *keys_in = (uint64_t *)(tmp + at_keys);
        int32_t *idx_in = (int32_t *)(tmp + at_idx);
        double *Htmp = (double *)(tmp + at_H);
        int64_t *width = (int64_t *)(tmp + at_width);
        void *work = tmp + at_work;

        // Morton order
        k_morton<<<nblk(n), kBlock, 0, st>>>(n, x, 1.0 / ctx->p.box, keys_in, idx_in);
        HIP_OR_FAIL(rocprim::radix_sort_pairs(work, sort_bytes, keys_in, ctx->keys, idx_in,
                                              ctx->perm32, (size_t)n, 0, 63, st));
        k_gather_sorted<<<nblk(n), kBlock, 0, st>>>(n, x, ctx->perm32, h_in, ctx->xs, h, perm);

        // tree on positions; smoothing lengths
        build_tree(ctx, nullptr);
        Tree T{ctx->node_lo, ctx->node_hi, ctx->node_hmax, ctx->P};
        const int depth = tree_depth(ctx);
        const int64_t n8 = (n + kPts - 1) / kPts;   // waves of the searches
        HIP_OR_FAIL(hipMemsetAsync(ctx->status, 0, sizeof(int32_t), st));
        if (!h_in) {
            k_h_guess<<<nblk(n), kBlock, 0, st>>>(n, ctx->P, ctx->node_lo, ctx->node_hi,
                                                  ctx->xs, ctx->p.eta, ctx->p.box, h);
            k_h_solve<<<(unsigned)xcd_grid(n8), 64, 0, st>>>(n, n8, T, depth, ctx->xs, ctx->p.eta,
                                                             ctx->p.kappa, ctx->p.box, h,
                                                             ctx->h_iter_cap, ctx->h_iters,
                                                             ctx->status);
            k_h_dense<<<(unsigned)std::min<int64_t>(xcd_grid(n8), kDenseGrid), 64, 0, st>>>(
                n, n8, T, depth, ctx->xs, ctx->p.eta, ctx->p.kappa, ctx->p.box, h, ctx->h_iter_cap,
                ctx->h_iters, ctx->status);
        } else {
            HIP_OR_FAIL(hipMemsetAsync(ctx->h_iters, 0, sizeof(int32_t) * n, st));
        }
        k_scale<<<nblk(n), kBlock, 0, st>>>(n, h, ctx->p.kappa, Htmp);
        build_tree(ctx, Htmp);
        // largest H must stay below half the box (nearest image is unique)
        int32_t stw = 0;
        double hmax = 0.0;
        HIP_OR_FAIL(hipMemcpyAsync(&stw, ctx->status, sizeof(int32_t), hipMemcpyDeviceToHost, st));
        HIP_OR_FAIL(hipMemcpyAsync(&hmax, ctx->node_hmax + 1, sizeof(double), hipMemcpyDeviceToHost, st));
        HIP_OR_FAIL(hipStreamSynchronize(st));
        if (stw & ST_NOCONV) { rs = rt_fail(ctx, RT_ENOCONV, "smoothing length did not converge"); goto fail; }
        if ((stw & ST_BIGH) || !(hmax < 0.5 * ctx->p.box)) {
            rs = rt_fail(ctx, RT_EINVAL, "compact support radius reaches half the box");
            goto fail;
        }
        // neighbour table: counts, wave widths, offsets, fill
        int ncap = (int)std::min<int64_t>(kNList, kNListBytes / (4 * n));
        if (ncap < kNList / 2 || !rt_try_alloc(ctx, (void **)&list_mem, sizeof(int32_t) * ncap * n)) {
            list_mem = nullptr;
            ncap = 0;
        }
        int32_t *nlist = (int32_t *)list_mem;
        k_neighbours_count<<<(unsigned)xcd_grid(n8), 64, 0, st>>>(n, n8, T, depth, ctx->xs, Htmp,
                                                                  ctx->p.box, ctx->n_nbr,
                                                                  ctx->n_gath, nlist, ncap);
        k_wave_width<<<nblk(nw + 1), kBlock, 0, st>>>(n, nw, ctx->n_nbr, width);
        HIP_OR_FAIL(rocprim::exclusive_scan(work, scan_bytes, width, ctx->wave_base, (int64_t)0,
                                            (size_t)(nw + 1), rocprim::plus<int64_t>(), st));
        int64_t locs = 0;                       // packed entries of a union
        HIP_OR_FAIL(hipMemcpyAsync(&ctx->slots, ctx->wave_base + nw, sizeof(int64_t),
                                   hipMemcpyDeviceToHost, st));
        if (ucap > 0) {
            k_union_width<<<nblk(nw + 1), kBlock, 0, st>>>(nw, ctx->wave_base, width);
            HIP_OR_FAIL(rocprim::exclusive_scan(work, scan_bytes, width, ctx->goff, (int64_t)0,
                                                (size_t)(nw + 1), rocprim::plus<int64_t>(), st));
            HIP_OR_FAIL(hipMemcpyAsync(&locs, ctx->goff + nw, sizeof(int64_t),
                                       hipMemcpyDeviceToHost, st));
        }
        HIP_OR_FAIL(hipStreamSynchronize(st));
        // (a little room, so that the next build's table, a few slots longer,
        // fits as well)
        const size_t slots = (size_t)std::max<int64_t>(ctx->slots, 1);
        if (!rt_holds(ctx, ctx->nbr, sizeof(int32_t) * slots))
            RESERVE(ctx->nbr, sizeof(int32_t) * (slots + slots / 64));
        if (!rt_holds(ctx, ctx->task, sizeof(int32_t) * slots))
            RESERVE(ctx->task, sizeof(int32_t) * (slots + slots / 64));
        if (ucap > 0 && !rt_holds(ctx, ctx->gloc, sizeof(uint16_t) * locs))
            RESERVE(ctx->gloc, sizeof(uint16_t) * (std::max<int64_t>(locs, 4) + locs / 64));
        if (acap > 0 && !rt_holds(ctx, ctx->agloc, sizeof(uint16_t) * locs))
            RESERVE(ctx->agloc, sizeof(uint16_t) * (std::max<int64_t>(locs, 4) + locs / 64));
        HIP_OR_FAIL(hipMemsetAsync(ctx->nbr, 0xff, sizeof(int32_t) * slots, st));
        k_neighbours_fill<<<nblk(n), kBlock, 0, st>>>(n, T, ctx->xs, Htmp, ctx->p.box, ctx->n_nbr,
                                                      ctx->n_gath, ctx->wave_base, ctx->nbr, nlist,
                                                      ncap);
        // task lists of the tile transports
        HIP_OR_FAIL(hipMemsetAsync(ctx->tstat, 0, 2 * sizeof(int64_t), st));
        k_tasks<<<(unsigned)nw, 64, 0, st>>>(n, ctx->wave_base, ctx->n_nbr, ctx->n_gath, ctx->nbr,
                                             ctx->task, ctx->n_task, ctx->tstat);
        // neighbour unions of the gradient (gather lists): FP64 at the 2-wave
        // capacity, then 3 waves per SIMD if nearly every block fits that
        // capacity; FP32C at its 3-wave capacity.  FP64 also builds those of
        // the adjoint's transposed gradient (the symmetric lists), which
        // stages one group at a time.
        if (ucap > 0) {
            k_union<<<(unsigned)xcd_grid(nw), 256, 0, st>>>(n, nw, ucap, ctx->wave_base, ctx->n_gath,
                                                            ctx->nbr, ctx->urows, ctx->urow,
                                                            ctx->goff, ctx->gloc, ctx->uown);
            k_union_left<<<1, 1024, 0, st>>>(nw, ctx->urows, f64 ? 2 : 3, ucap3, ctx->ublk);
        }
        if (acap > 0) {
            k_union<<<(unsigned)xcd_grid(nw), 256, 0, st>>>(n, nw, acap, ctx->wave_base, ctx->n_nbr,
                                                            ctx->nbr, ctx->arows, ctx->arow,
                                                            ctx->goff, ctx->agloc, ctx->aown);
            k_union_left<<<1, 1024, 0, st>>>(nw, ctx->arows, 2, adj_union_cap(3), ctx->ablk);
        }
        // geometry records, volumes, time step, statistics
        HIP_OR_FAIL(hipMemsetAsync(ctx->status, 0, sizeof(int32_t), st));
        HIP_OR_FAIL(hipMemsetAsync(ctx->result, 0, sizeof(BuildResult), st));
        k_geometry<<<nblk(n), kBlock, 0, st>>>(n, ctx->xs, h, ctx->p.kappa, ctx->p.box,
                                               ctx->n_gath, ctx->wave_base, ctx->nbr, ctx->geo,
                                               ctx->geo32, V, ctx->vol, ctx->dxpart, ctx->status);
        k_dt<<<1, kBlock, 0, st>>>(nblk(n), ctx->dxpart, ctx->p.cfl, ctx->p.c_red, ctx->dt_dev);
        if (dt) k_copy_dt<<<1, 1, 0, st>>>(ctx->dt_dev, dt);
        k_stats<<<std::min<unsigned>(nblk(n), 128), kBlock, 0, st>>>(n, ctx->n_nbr, ctx->n_gath,
                                                                      ctx->h_iters, ctx->result);
        k_result<<<1, 1, 0, st>>>(ctx->status, ucap > 0 ? ctx->ublk : nullptr,
                                  acap > 0 ? ctx->ablk : nullptr, ctx->result);
        HIP_OR_FAIL(hipGetLastError());
        HIP_OR_FAIL(hipMemcpyAsync(&res, ctx->result, sizeof res, hipMemcpyDeviceToHost, st));
        HIP_OR_FAIL(hipStreamSynchronize(st));
        if (res.status & ST_SINGULAR) {
            rs = rt_fail(ctx, RT_ESINGULAR, "E_i not positive definite (coplanar or too few neighbours)");
            goto fail;
        }
    }
    ctx->n_entries = (int64_t)res.stat[0];
    ctx->n_gather_entries = (int64_t)res.stat[1];
    ctx->h_list_overflow = (int64_t)res.stat[2];
    ctx->max_nbr = (int32_t)res.stat[3];
    ctx->h_iter_max = (int32_t)res.stat[4];
    ctx->n_ublk = res.left[0];
    ctx->union_waves = res.left[1];
    ctx->n_ablk = res.aleft[0];
    ctx->adj_union_waves = res.aleft[1];
    // larger unions for the few blocks over the capacity
    ctx->n_lblk = 0;
    ctx->n_sblk = ctx->n_ublk;
    ctx->sblk = ctx->n_ublk > 0 ? ctx->ublk + 2 : nullptr;
    if (ucap > 0 && union_cap_large(G) > ucap && ctx->n_ublk > 0 &&
        ctx->n_ublk <= large_blocks(f64)) {
        const int64_t most = large_blocks(f64);
        const int64_t nl = ctx->n_ublk;
        const int lcap = union_cap_large(G);
        int32_t left = 0;
        RESERVE(ctx->lrows, sizeof(int32_t) * most);
        RESERVE(ctx->lrow, sizeof(int32_t) * most * lcap);
        RESERVE(ctx->lblk, sizeof(int32_t) * (most + 2));
        k_union<<<(unsigned)xcd_grid(nl), 256, 0, st>>>(n, nl, lcap, ctx->wave_base, ctx->n_gath,
                                                        ctx->nbr, ctx->lrows, ctx->lrow, ctx->goff,
                                                        ctx->gloc, ctx->uown, ctx->ublk + 2);
        k_union_left<<<1, 1024, 0, st>>>(nl, ctx->lrows, 1, 0, ctx->lblk, ctx->ublk + 2);
        HIP_OR_FAIL(hipGetLastError());
        HIP_OR_FAIL(hipMemcpyAsync(&left, ctx->lblk, sizeof left, hipMemcpyDeviceToHost, st));
        HIP_OR_FAIL(hipStreamSynchronize(st));
        ctx->n_lblk = nl;
        ctx->n_sblk = left;
        ctx->sblk = ctx->lblk + 2;
    }
    rt_free(ctx, list_mem);
    if ((rs = rt_ensure_partials(ctx)) != RT_OK) return rs;
    ctx->built = 1;
    if (ctx->surfaces == RT_IVANOVA && (rs = rt_ivanova_impl(ctx)) != RT_OK) return rs;
    ctx->bin_top = -1;   // the records were rewritten with all time bins 0
    if (ctx->bin8) RT_HIP(hipMemsetAsync(ctx->bin8, 0, 2 * (size_t)n, st));
    return RT_OK;
fail:
    // the conditions of the build are reported by its return code, not by a
    // later rt_sync
    (void)hipMemsetAsync(ctx->status, 0, sizeof(int32_t), st);
    (void)hipStreamSynchronize(st);
    rt_free(ctx, list_mem);
    return rs;
#undef RESERVE
#undef HIP_OR_FAIL
}

rt_status rt_sources_impl(rt_ctx *ctx, int32_t S, const double *xs, double eta_star) {
    hipStream_t st = ctx->stream;
    rt_free(ctx, ctx->src_h); rt_free(ctx, ctx->inj_gptr); rt_free(ctx, ctx->inj_gas); rt_free(ctx, ctx->inj_src);
    rt_free(ctx, ctx->inj_coef); rt_free(ctx, ctx->inj_xi); rt_free(ctx, ctx->src_ptr); rt_free(ctx, ctx->src_gas);
    rt_free(ctx, ctx->src_coef);
    ctx->src_h = nullptr; ctx->inj_gptr = nullptr; ctx->inj_gas = nullptr; ctx->inj_src = nullptr;
    ctx->inj_coef = nullptr; ctx->inj_xi = nullptr; ctx->src_ptr = nullptr; ctx->src_gas = nullptr;
    ctx->src_coef = nullptr;
    ctx->S = 0;
    ctx->n_inj = 0;
    ctx->n_inj_gas = 0;
    if (S == 0) return RT_OK;
    const int64_t n = ctx->p.n;
    rt_status rs;
    double *sx = nullptr, *sxi = nullptr;
    int32_t *cnt = nullptr;
    std::vector<int32_t> hc(S), hptr(S + 1);
    Tree T{ctx->node_lo, ctx->node_hi, ctx->node_hmax, ctx->P};
    if ((rs = rt_alloc(ctx, (void **)&sx, sizeof(double) * 3 * S)) != RT_OK) return rs;
    if ((rs = rt_alloc(ctx, (void **)&ctx->src_h, sizeof(double) * S)) != RT_OK) goto fail;
    if ((rs = rt_alloc(ctx, (void **)&cnt, sizeof(int32_t) * S)) != RT_OK) goto fail;
    RT_HIP(hipMemcpyAsync(sx, xs, sizeof(double) * 3 * S, hipMemcpyDeviceToDevice, st));
    RT_HIP(hipMemsetAsync(ctx->status, 0, sizeof(int32_t), st));
    {
        const int depth = tree_depth(ctx);
        k_src_h<<<(unsigned)S, 64, 0, st>>>(S, T, depth, ctx->xs, n, ctx->keys, ctx->geo, sx,
                                            eta_star, ctx->p.kappa, ctx->p.box, ctx->h_iter_cap,
                                            ctx->src_h, ctx->status);
        k_src_gas<false><<<(unsigned)S, 64, 0, st>>>(S, T, depth, ctx->xs, n, sx, ctx->src_h,
                                                     ctx->p.kappa, ctx->p.box, ctx->geo, cnt,
                                                     nullptr, nullptr, nullptr, nullptr);
        int32_t stw = 0;
        RT_HIP(hipMemcpyAsync(hc.data(), cnt, sizeof(int32_t) * S, hipMemcpyDeviceToHost, st));
        RT_HIP(hipMemcpyAsync(&stw, ctx->status, sizeof(int32_t), hipMemcpyDeviceToHost, st));
        RT_HIP(hipStreamSynchronize(st));
        if (stw & ST_NOCONV) { rs = rt_fail(ctx, RT_ENOCONV, "source smoothing length did not converge"); goto fail; }
        if (stw & ST_BIGH) { rs = rt_fail(ctx, RT_EINVAL, "source compact support reaches half the box"); goto fail; }
        hptr[0] = 0;
        for (int32_t s = 0; s < S; ++s) {
            if (hc[s] == 0) { rs = rt_fail(ctx, RT_EINVAL, "source without gas neighbours"); goto fail; }
            hptr[s + 1] = hptr[s] + hc[s];
        }
        const int64_t m = hptr[S];
        if ((rs = rt_alloc(ctx, (void **)&ctx->src_ptr, sizeof(int32_t) * (S + 1))) != RT_OK) goto fail;
        if ((rs = rt_alloc(ctx, (void **)&ctx->src_gas, sizeof(int32_t) * m)) != RT_OK) goto fail;
        if ((rs = rt_alloc(ctx, (void **)&ctx->src_coef, sizeof(double) * m)) != RT_OK) goto fail;
        if ((rs = rt_alloc(ctx, (void **)&sxi, sizeof(double) * m)) != RT_OK) goto fail;
        RT_HIP(hipMemcpyAsync(ctx->src_ptr, hptr.data(), sizeof(int32_t) * (S + 1),
                              hipMemcpyHostToDevice, st));
        k_src_gas<true><<<(unsigned)S, 64, 0, st>>>(S, T, tree_depth(ctx), ctx->xs, n, sx,
                                                   ctx->src_h, ctx->p.kappa, ctx->p.box, ctx->geo, nullptr, ctx->src_ptr,
                                                   ctx->src_gas, sxi, ctx->src_coef);
        // gas-major copy for the per-step injection (deterministic gather)
        std::vector<int32_t> g(m), srcv(m);
        std::vector<double> xi(m), co(m);
        RT_HIP(hipMemcpyAsync(g.data(), ctx->src_gas, sizeof(int32_t) * m, hipMemcpyDeviceToHost, st));
        RT_HIP(hipMemcpyAsync(xi.data(), sxi, sizeof(double) * m, hipMemcpyDeviceToHost, st));
        RT_HIP(hipMemcpyAsync(co.data(), ctx->src_coef, sizeof(double) * m, hipMemcpyDeviceToHost, st));
        RT_HIP(hipStreamSynchronize(st));
        for (int32_t s = 0; s < S; ++s)
            for (int32_t e = hptr[s]; e < hptr[s + 1]; ++e) srcv[e] = s;
        std::vector<int64_t> ord(m);
        std::iota(ord.begin(), ord.end(), 0);
        std::stable_sort(ord.begin(), ord.end(), [&](int64_t a, int64_t b) { return g[a] < g[b]; });
        std::vector<int32_t> ig, igp, isr(m);
        std::vector<double> ico(m), ixi(m);
        for (int64_t e = 0; e < m; ++e) {
            int64_t o = ord[e];
            if (e == 0 || g[o] != g[ord[e - 1]]) {
                ig.push_back(g[o]);
                igp.push_back((int32_t)e);
            }
            isr[e] = srcv[o];
            ico[e] = co[o];
            ixi[e] = xi[o];
        }
        igp.push_back((int32_t)m);
        ctx->n_inj = m;
        ctx->n_inj_gas = (int32_t)ig.size();
        if ((rs = rt_alloc(ctx, (void **)&ctx->inj_gptr, sizeof(int32_t) * igp.size())) != RT_OK) goto fail;
        if ((rs = rt_alloc(ctx, (void **)&ctx->inj_gas, sizeof(int32_t) * ig.size())) != RT_OK) goto fail;
        if ((rs = rt_alloc(ctx, (void **)&ctx->inj_src, sizeof(int32_t) * m)) != RT_OK) goto fail;
        if ((rs = rt_alloc(ctx, (void **)&ctx->inj_coef, sizeof(double) * m)) != RT_OK) goto fail;
        if ((rs = rt_alloc(ctx, (void **)&ctx->inj_xi, sizeof(double) * m)) != RT_OK) goto fail;
        RT_HIP(hipMemcpyAsync(ctx->inj_gptr, igp.data(), sizeof(int32_t) * igp.size(), hipMemcpyHostToDevice, st));
        RT_HIP(hipMemcpyAsync(ctx->inj_gas, ig.data(), sizeof(int32_t) * ig.size(), hipMemcpyHostToDevice, st));
        RT_HIP(hipMemcpyAsync(ctx->inj_src, isr.data(), sizeof(int32_t) * m, hipMemcpyHostToDevice, st));
        RT_HIP(hipMemcpyAsync(ctx->inj_coef, ico.data(), sizeof(double) * m, hipMemcpyHostToDevice, st));
        RT_HIP(hipMemcpyAsync(ctx->inj_xi, ixi.data(), sizeof(double) * m, hipMemcpyHostToDevice, st));
        RT_HIP(hipStreamSynchronize(st));
    }
    ctx->S = S;
    rt_free(ctx, sx); rt_free(ctx, cnt); rt_free(ctx, sxi);
    return RT_OK;
fail:
    (void)hipMemsetAsync(ctx->status, 0, sizeof(int32_t), st);
    (void)hipStreamSynchronize(st);
    rt_free(ctx, sx); rt_free(ctx, cnt); rt_free(ctx, sxi);
    return rs;
}
