// Per-step kernels of the photon transport (Part III "One RT time step"):
// injection, least-squares gradients, the pair transport loop with its fused
// update, and the photon budget.
//
// Every kernel is a gather over the wave-sliced neighbour table: lane i owns
// particle i (Morton order), reads slot j of its list at
// wave_base[i/64] + 64 j + i%64 (coalesced), and accumulates in registers, so
// results are deterministic and no atomics touch floating-point state.
#include "rt_pair.h"

using namespace gearrt;

namespace {

inline unsigned nblk(int64_t n, int b = kBlock) { return (unsigned)((n + b - 1) / b); }

// ---------------------------------------------------------------------------
// Injection: E_g += dt sum_s xi_sg L_s / V_g, one thread per receiving particle.
template <typename T>
__global__ void k_inject(int32_t ngas, int G, const int32_t *__restrict__ gptr,
                         const int32_t *__restrict__ gas, const int32_t *__restrict__ src,
                         const double *__restrict__ coef, const double *__restrict__ L,
                         const double *__restrict__ dtp, T *__restrict__ U) {
    int32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= ngas) return;
    const int64_t g = gas[t];
    const double dt = dtp[0];
    for (int grp = 0; grp < G; ++grp) {
        double s = 0.0;
        for (int32_t e = gptr[t]; e < gptr[t + 1]; ++e) s += coef[e] * L[(int64_t)src[e] * G + grp];
        T *E = U + (g * G + grp) * 4;
        E[0] = (T)((double)E[0] + dt * s);
    }
}

// Gradient record of particle i from its Q lanes' sums (every lane holds the
// combined sums acc = sum_j (q_j - q_i) w_ij s_ij and the own state Ui): the
// gradients are B_i/V_i acc; the Q lanes write consecutive 16-byte pieces of
// the record.  chk stays 0 unless a value written is NaN or infinite (0 x v is
// 0 for finite v and NaN otherwise).
template <int G, int Q>
__device__ __forceinline__ void gradient_record(double (&acc)[4 * G][3], const double (&Ui)[4 * G],
                                                const double *__restrict__ rec, double *o, int sub,
                                                int32_t *__restrict__ status) {
    constexpr int NQ = 4 * G;
    const double iV = 1.0 / rec[R_V];
    const double b00 = rec[R_B] * iV, b01 = rec[R_B + 1] * iV, b02 = rec[R_B + 2] * iV;
    const double b11 = rec[R_B + 3] * iV, b12 = rec[R_B + 4] * iV, b22 = rec[R_B + 5] * iV;
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
        const double d0 = b00 * acc[q][0] + b01 * acc[q][1] + b02 * acc[q][2];
        const double d1 = b01 * acc[q][0] + b11 * acc[q][1] + b12 * acc[q][2];
        const double d2 = b02 * acc[q][0] + b12 * acc[q][1] + b22 * acc[q][2];
        acc[q][0] = d0;
        acc[q][1] = d1;
        acc[q][2] = d2;
    }
    // group-major record: per group the state then its gradients (one line);
    // double d of the record, d = 16 g + s
    auto value = [&](int d) {
        const int g = d / 16, s = d % 16;
        return s < 4 ? Ui[4 * g + s] : acc[4 * g + (s - 4) / 3][(s - 4) % 3];
    };
    double chk = 0.0;
#pragma unroll
    for (int t = 0; t < 8 * G / Q; ++t) {
        double2 val = make_double2(value(2 * Q * t), value(2 * Q * t + 1));
#pragma unroll
        for (int s = 1; s < Q; ++s)
            if (sub == s) val = make_double2(value(2 * (Q * t + s)), value(2 * (Q * t + s) + 1));
        chk = __builtin_fma(val.x, 0.0, chk);
        chk = __builtin_fma(val.y, 0.0, chk);
        *reinterpret_cast<double2 *>(o + 2 * (Q * t + sub)) = val;
    }
    if (chk != chk) atomicOr(status, ST_NONFINITE);
}

// Reduce-scatter of a particle's four lanes' partial sums (4 lanes a
// particle, DPP): afterwards lane sub holds in s[g] the full sums of
// component sub of every group g, formed with the same additions in the same
// order as quad_sum, so with the same bits, while no lane holds all 12 G sums
// (the record then needs a quarter of the registers).  After the first step
// slot k of a lane with bit 0 = b0 holds q = 2k + b0, after the second slot g
// of lane sub holds q = 4g + sub.
template <int G>
__device__ __forceinline__ void quad_scatter(const double (&acc)[4 * G][3], int sub,
                                             double (&s)[G][3]) {
    const bool b0 = (sub & 1) != 0, b1 = (sub & 2) != 0;
    double t[2 * G][3];
#pragma unroll
    for (int k = 0; k < 2 * G; ++k)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const double mine = b0 ? acc[2 * k + 1][a] : acc[2 * k][a];
            const double other = b0 ? acc[2 * k][a] : acc[2 * k + 1][a];
            t[k][a] = mine + quad_xor<1>(other);
        }
#pragma unroll
    for (int g = 0; g < G; ++g)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const double mine = b1 ? t[2 * g + 1][a] : t[2 * g][a];
            const double other = b1 ? t[2 * g][a] : t[2 * g + 1][a];
            s[g][a] = mine + quad_xor<2>(other);
        }
}

// The record from the scattered sums (gradient_record's arithmetic): lane sub
// writes component sub of every group, its state u[g] and its gradient.
template <int G>
__device__ __forceinline__ void gradient_record_part(const double (&s)[G][3], const double (&u)[G],
                                                     const double *__restrict__ rec, double *o,
                                                     int sub, int32_t *__restrict__ status) {
    const double iV = 1.0 / rec[R_V];
    const double b00 = rec[R_B] * iV, b01 = rec[R_B + 1] * iV, b02 = rec[R_B + 2] * iV;
    const double b11 = rec[R_B + 3] * iV, b12 = rec[R_B + 4] * iV, b22 = rec[R_B + 5] * iV;
    double chk = 0.0;
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const double d0 = b00 * s[g][0] + b01 * s[g][1] + b02 * s[g][2];
        const double d1 = b01 * s[g][0] + b11 * s[g][1] + b12 * s[g][2];
        const double d2 = b02 * s[g][0] + b12 * s[g][1] + b22 * s[g][2];
        double *og = o + 16 * g;
        og[sub] = u[g];
        og[4 + 3 * sub] = d0;
        og[5 + 3 * sub] = d1;
        og[6 + 3 * sub] = d2;
        chk = __builtin_fma(u[g], 0.0, chk);
        chk = __builtin_fma(d0, 0.0, chk);
        chk = __builtin_fma(d1, 0.0, chk);
        chk = __builtin_fma(d2, 0.0, chk);
    }
    if (chk != chk) atomicOr(status, ST_NONFINITE);
}

// ---------------------------------------------------------------------------
// Gradient (eq:gradient):  grad q_i = sum_j (q_j - q_i) psi~_j(x_i)
//   = S_i^{-1} sum_j (q_j - q_i) w(r_ij / H_i) s_ij   (the kernel normalisation
// and V_i cancel against B_i, see the geometry record).
// BIN: only the particles that end a step in tick `tick` (time bin in slot 12
// of the geometry record) recompute their gradient record.
//
// Q lanes share a particle, each summing every Q-th gather neighbour; the
// partial sums are combined by a fixed butterfly (the same bits on every lane
// of the particle), and the Q lanes write the particle's record together.
//
// Neighbour rows are staged through LDS.  Gathered lane by lane, each of the
// 8 loads of a neighbour's state and position touches 64 different cache
// lines (1.31 ms on the 3-group 128^3 lattice, the L1 doing about one tag
// lookup a cycle).  Here the wave moves the 64 rows of an iteration with
// consecutive lanes taking consecutive pieces: 2G loads of 16 bytes for the
// neighbours' states (64 / 2G rows a load) and 3 of 8 bytes for their
// positions (x, y, z from the packed position array, 21 rows a load; the
// heads of the 128-byte geometry records would take a cache line per
// neighbour and raised the L1 misses by 60%).  The lane that stores a piece
// subtracts the same piece of the row's own particle (the wave's own rows sit
// in LDS in the same layout), so a lane reads U_j - U_i and x_j - x_i from its
// row and holds neither its own state nor its position, which keeps the
// kernel at 3 waves per SIMD without spills.  State rows lie 2G + 1 pieces of
// 16 bytes apart in LDS, an odd number, and positions are packed 3 doubles a
// row in an array of their own, so that the stores and reads of both are
// free of bank conflicts (8-byte halves of the state pieces, or positions
// inside the state rows, conflicted 2-way).  Past
// the end of its list a lane's row is its own particle's, whose differences
// are zero: the sums need no branch.  The table entry of an iteration is
// loaded two iterations ahead and its rows one.  1.20 ms on the lattice: the
// texture data path stays busy 95% of the time, half of it waiting for L1
// misses (a wave's 16 particles reach about 400 distinct neighbours, more
// than the L1 holds).  Two iterations of rows in flight at 2 waves per SIMD
// ran 1.25 ms, blocks of 8 and 12 waves 1.41 and 1.31 ms.
#ifndef RT_GRADIENT_WAVES
#define RT_GRADIENT_WAVES 3
#endif
#ifndef RT_GRADIENT_BLOCK
#define RT_GRADIENT_BLOCK 4
#endif
constexpr int gradient_waves(int G) { return G <= 3 ? RT_GRADIENT_WAVES : G == 4 ? 2 : 1; }
static_assert(RT_GRADIENT_BLOCK >= 1 && RT_GRADIENT_BLOCK <= 16, "1 to 16 waves per block");
// threads per block of the FP64 gradient: at most the waves of one CU and
// the LDS of one CU (80 staged rows of 2G + 1 pieces and 3 doubles per wave at
// 4 lanes per particle)
constexpr int grad_lds_wave(int G) { return 80 * ((2 * G + 1) * 16 + 24); }
constexpr int grad_block(int G) {
    const int by_lds = 163840 / grad_lds_wave(G);
    int w = RT_GRADIENT_BLOCK;
    if (w > 4 * gradient_waves(G)) w = 4 * gradient_waves(G);
    if (w > by_lds) w = by_lds;
    return 64 * w;
}

template <int G, bool BIN = false, int Q = 1>
__global__ __launch_bounds__(grad_block(G)) __attribute__((amdgpu_waves_per_eu(
    gradient_waves(G), gradient_waves(G)))) void k_gradient64(
    int64_t n, int64_t nb, const double *__restrict__ geo, const double *__restrict__ xs,
    const int32_t *__restrict__ nbr, const int64_t *__restrict__ wave_base,
    const int32_t *__restrict__ n_gath, const double *__restrict__ U, double *__restrict__ UD,
    int32_t *__restrict__ status, double box, int64_t tick = 0,
    const int32_t *__restrict__ blist = nullptr) {
    static_assert(Q == 1 || Q == 2 || Q == 4, "lanes per particle: 1, 2 or 4");
    constexpr int NQ = 4 * G;
    constexpr int PU = 2 * G;           // 16-byte pieces of a state
    constexpr int S = PU + 1;           // LDS row stride in pieces (odd)
    constexpr int NP = 64 / Q;          // particles of a wave
    constexpr int W = grad_block(G) / 64;
    static_assert(Q != 4 || grad_lds_wave(G) * W <= 163840, "LDS of one CU");
    __shared__ dvec2 stage[W][64 * S];
    __shared__ dvec2 own[W][NP * S];
    __shared__ double spos[W][64 * 3];
    __shared__ double opos[W][NP * 3];
    const int64_t bx = xcd_block(nb);
    if (bx >= nb) return;                       // whole block
    const int64_t blk = blist ? (int64_t)blist[bx] : bx;   // only the listed blocks
    const int lane = threadIdx.x & 63;
    const int sub = lane % Q;
    // the wave's first particle; the wave stays whole (its loads are shared)
    const int64_t i0 = blk * (grad_block(G) / Q) + (threadIdx.x >> 6) * NP;
    if (i0 >= n) return;                        // whole wave
    const int64_t i = i0 + lane / Q;
    const int64_t ic = i < n ? i : n - 1;
    const double *rec = geo + (int64_t)kRec * ic;
    const bool active =
        i < n && (!BIN || ((tick + 1) & ((int64_t(1) << (int32_t)rec[12]) - 1)) == 0);
    const int32_t ng = active ? n_gath[ic] : 0;
    int32_t kmax = ng;                          // the wave's longest list
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) kmax = max(kmax, __shfl_xor(kmax, o, 64));
    const double ibox = 1.0 / box;
    const double iH = rec[R_IH];
    double acc[NQ][3];
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc[q][0] = acc[q][1] = acc[q][2] = 0.0;
    dvec2 *sb = stage[threadIdx.x >> 6], *ob = own[threadIdx.x >> 6];
    double *sd = spos[threadIdx.x >> 6], *od = opos[threadIdx.x >> 6];
    const dvec2 *U2 = reinterpret_cast<const dvec2 *>(U);
    // the wave's own rows (the last particle repeated past n)
#pragma unroll
    for (int c = 0; c < (NP * PU + 63) / 64; ++c) {
        const int e = 64 * c + lane;
        if (NP * PU % 64 == 0 || e < NP * PU) {
            const uint32_t jo = (uint32_t)min(i0 + e / PU, n - 1);
            ob[(e / PU) * S + e % PU] = U2[jo * (uint32_t)PU + (uint32_t)(e % PU)];
        }
    }
#pragma unroll
    for (int c = 0; c < (NP * 3 + 63) / 64; ++c) {
        const int e = 64 * c + lane;
        if (NP * 3 % 64 == 0 || e < NP * 3) {
            const uint32_t jo = (uint32_t)min(i0 + e / 3, n - 1);
            od[e] = xs[jo * 3u + (uint32_t)(e % 3)];
        }
    }
    if (kmax > 0) {
        // Slot k of the particle's column, or slot 0 past the end of its list
        // (present: some column of this table block holds an entry); an index
        // past the end is replaced by the particle's own.
        const int32_t *col = nbr + wave_base[ic >> 6] + (ic & 63);
        auto entry = [&](int32_t k) __attribute__((always_inline)) {
            return col[64 * (k < ng ? k : 0)];
        };
        auto index = [&](int32_t k, int32_t e) __attribute__((always_inline)) {
            return k < ng ? e : (int32_t)ic;
        };
        // the rows of lane j's: state piece c of every lane is e = 64 c + lane,
        // row e / PU; position double c is e = 64 c + lane, row e / 3
        struct Rows { dvec2 u[PU]; double x[3]; };
        auto load = [&](Rows &v, int32_t j) __attribute__((always_inline)) {
#pragma unroll
            for (int c = 0; c < PU; ++c) {
                const int e = 64 * c + lane;
                const uint32_t jr = (uint32_t)__shfl(j, e / PU, 64);
                v.u[c] = U2[jr * (uint32_t)PU + (uint32_t)(e % PU)];
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const int e = 64 * c + lane;
                const uint32_t jr = (uint32_t)__shfl(j, e / 3, 64);
                v.x[c] = xs[jr * 3u + (uint32_t)(e % 3)];
            }
        };
        // store the pieces less the own particle's, for the lanes to read
        auto put = [&](const Rows &v) __attribute__((always_inline)) {
            wave_lds_sync();
#pragma unroll
            for (int c = 0; c < PU; ++c) {
                const int e = 64 * c + lane, r = e / PU, p = e % PU;
                sb[r * S + p] = v.u[c] - ob[(r / Q) * S + p];
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const int e = 64 * c + lane;
                sd[e] = v.x[c] - od[(e / (3 * Q)) * 3 + e % 3];
            }
            wave_lds_sync();
        };
        auto gather = [&]() __attribute__((always_inline)) {
            const dvec2 *row = sb + lane * S;
            const double sx = min_image(sd[3 * lane], box, ibox);
            const double sy = min_image(sd[3 * lane + 1], box, ibox);
            const double sz = min_image(sd[3 * lane + 2], box, ibox);
            const double w = kern_w(sqrt64(sx * sx + sy * sy + sz * sz) * iH);
            const double wx = w * sx, wy = w * sy, wz = w * sz;
#pragma unroll
            for (int t = 0; t < PU; ++t) {
                const dvec2 d = row[t];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int q = 2 * t + h;
                    acc[q][0] += d[h] * wx;
                    acc[q][1] += d[h] * wy;
                    acc[q][2] += d[h] * wz;
                }
            }
        };
        // Each table entry is loaded before the rows of the iteration ahead of
        // it, so waiting for the entry never waits for rows still in flight;
        // no step is skipped near the end (rows past every list are the own
        // rows), so that every path through the loop body is alike.
        Rows v;
        const int32_t e0 = entry(sub);
        int32_t e1 = entry(Q + sub);
        load(v, index(sub, e0));
        for (int32_t kk = 0; kk < kmax; kk += Q) {
            put(v);
            const int32_t e2 = entry(kk + 2 * Q + sub);
            load(v, index(kk + Q + sub, e1));
            e1 = e2;
            gather();
        }
    }
    if constexpr (Q == 4) {
        double sg[G][3];
        quad_scatter<G>(acc, sub, sg);
        if (!active) return;
        // the own state, as loaded, from the wave's own row: component sub
        wave_lds_sync();
        double u[G];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const dvec2 x = ob[(lane / Q) * S + 2 * g + (sub >> 1)];
            u[g] = (sub & 1) ? x.y : x.x;
        }
        gradient_record_part<G>(sg, u, rec, UD + ic * (16 * G), sub, status);
        return;
    }
    if (Q > 1) {
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int a = 0; a < 3; ++a)
                quad_sum<Q>(acc[q][a]);
    }
    if (!active) return;
    // the own state, as loaded, from the wave's own row
    wave_lds_sync();
    double Ui[NQ];
#pragma unroll
    for (int t = 0; t < PU; ++t) {
        const dvec2 x = ob[(lane / Q) * S + t];
        Ui[2 * t] = x.x;
        Ui[2 * t + 1] = x.y;
    }
    gradient_record<G, Q>(acc, Ui, rec, UD + ic * (16 * G), sub, status);
}

// Gradient from the block's neighbour union (FP64, up to 4 groups, the global
// step).  The 64 particles of a block (a column block of the neighbour table)
// gather from about 360 (lattice) to 580 (Plummer set) distinct particles,
// each 6-8 times.  The build lists them (k_union); this kernel stages their
// states and positions in LDS once, with coalesced loads, and every pair then
// reads its neighbour's row from LDS by its 16-bit position in the union
// (gloc): the pair loop's only global loads are the table's entries, 8 bytes
// per 4 iterations.
// W = 1: larger unions, one block to a CU, of the blocks listed in blist (in
// its order: urows, urow), if they are few (large_blocks).  Blocks whose union
// fits neither are left to k_gradient64, by list.  Sums in the same order as k_gradient64 (lane sub
// takes the slots sub, sub + Q, ...; rows past a list are the own row, whose
// differences are zero), so the two give the same bits.
// BIN: only the particles that end a step in tick `tick` recompute their
// record, as in k_gradient64; a block none of whose particles does so stages
// nothing.
template <int G, int Q, int W, bool BIN = false>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(W, W))) void
k_gradient64u(int64_t n, int64_t nb, const double *__restrict__ geo, const double *__restrict__ xs,
              const int32_t *__restrict__ urow, const int32_t *__restrict__ urows,
              const uint16_t *__restrict__ gloc, const int64_t *__restrict__ goff,
              const uint16_t *__restrict__ uown, const int32_t *__restrict__ n_gath,
              const double *__restrict__ U, double *__restrict__ UD, int32_t *__restrict__ status,
              double box, int64_t tick = 0, const int32_t *__restrict__ blist = nullptr) {
    static_assert(Q == 4 && kBlock == 256, "one block of 64 particles per table column block");
    constexpr int UR = W == 1 ? union_cap_large(G) : union_cap(G);   // stride of the rows
    constexpr int NQ = 4 * G, PU = 2 * G, UC = W == 3 ? union_cap3(G) : UR;
    static_assert(UC > 0 && UC <= kUnionSort, "union capacity");
    __shared__ dvec2 ust[UC * PU];
    __shared__ double upos[UC * 3];
    __shared__ int32_t uidx[UC];
    const int64_t bx = xcd_block(nb);
    if (bx >= nb) return;                       // whole block
    const int64_t blk = W == 1 ? (int64_t)blist[bx] : bx;
    const int64_t u0 = bx * UR;
    const int32_t rows = urows[bx];
    if (rows == 0 || rows > UC) return;                      // left to the staged gradient (whole block)
    if constexpr (BIN) {
        const int64_t ib = blk * (kBlock / Q) + threadIdx.x / Q;
        const bool e = ib < n &&
                       ((tick + 1) & ((int64_t(1) << (int32_t)geo[(int64_t)kRec * ib + 12]) - 1)) == 0;
        if (!__syncthreads_or(e)) return;       // whole block: no particle ends a step
    }
    // stage the union: its indices first, then every thread's pieces of the
    // states (16 bytes) and positions (doubles) in flight at once (a chain of
    // dependent loads per piece left the blocks waiting: 1.38 ms)
    for (int e = threadIdx.x; e < rows; e += kBlock) uidx[e] = urow[u0 + e];
    __syncthreads();
    const dvec2 *U2 = reinterpret_cast<const dvec2 *>(U);
    const int ts = rows * PU, tp = rows * 3;
    {
        constexpr int MS = (UC * PU + kBlock - 1) / kBlock, MP = (UC * 3 + kBlock - 1) / kBlock;
        dvec2 v[MS];
        double x[MP];
#pragma unroll
        for (int r = 0; r < MS; ++r) {
            const int e = threadIdx.x + r * kBlock;
            if (e < ts) v[r] = U2[(uint32_t)uidx[e / PU] * (uint32_t)PU + (uint32_t)(e % PU)];
        }
#pragma unroll
        for (int r = 0; r < MP; ++r) {
            const int e = threadIdx.x + r * kBlock;
            if (e < tp) x[r] = xs[(uint32_t)uidx[e / 3] * 3u + (uint32_t)(e % 3)];
        }
#pragma unroll
        for (int r = 0; r < MS; ++r)
            if (threadIdx.x + r * kBlock < ts) ust[threadIdx.x + r * kBlock] = v[r];
#pragma unroll
        for (int r = 0; r < MP; ++r)
            if (threadIdx.x + r * kBlock < tp) upos[threadIdx.x + r * kBlock] = x[r];
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, sub = lane % Q;
    const int p = threadIdx.x / Q;              // the particle in the block
    const int64_t i = blk * (kBlock / Q) + p;
    const bool active =
        i < n && (!BIN || ((tick + 1) & ((int64_t(1) << (int32_t)geo[(int64_t)kRec * i + 12]) - 1)) == 0);
    const int64_t ic = active ? i : n - 1;
    const int32_t ng = active ? n_gath[ic] : 0;
    const int il = active ? (int)uown[ic] : 0;  // a row of the union (not used past n)
    int32_t kmax = ng;                          // the wave's longest list
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) kmax = max(kmax, __shfl_xor(kmax, o, 64));
    const double *rec = geo + (int64_t)kRec * ic;
    const double ibox = 1.0 / box, iH = rec[R_IH];
    double Ui[NQ];
#pragma unroll
    for (int t = 0; t < PU; ++t) {
        const dvec2 x = ust[il * PU + t];
        Ui[2 * t] = x.x;
        Ui[2 * t + 1] = x.y;
    }
    const double px = upos[3 * il], py = upos[3 * il + 1], pz = upos[3 * il + 2];
    double acc[NQ][3];
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc[q][0] = acc[q][1] = acc[q][2] = 0.0;
    if (kmax > 0) {
        auto pair = [&](int jl) __attribute__((always_inline)) {
            const dvec2 *row = ust + jl * PU;
            const double sx = min_image(upos[3 * jl] - px, box, ibox);
            const double sy = min_image(upos[3 * jl + 1] - py, box, ibox);
            const double sz = min_image(upos[3 * jl + 2] - pz, box, ibox);
            const double w = kern_w(sqrt64(sx * sx + sy * sy + sz * sz) * iH);
            const double wx = w * sx, wy = w * sy, wz = w * sz;
#pragma unroll
            for (int t = 0; t < PU; ++t) {
                const dvec2 uj = row[t];
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const int q = 2 * t + h;
                    const double d = uj[h] - Ui[q];
                    acc[q][0] += d * wx;
                    acc[q][1] += d * wy;
                    acc[q][2] += d * wz;
                }
            }
        };
        // The lane's table entries come packed 4 iterations to an 8-byte word
        // (group gq of the block's words at gw + 256 gq), each word loaded a
        // group pair ahead into the register its own use has just freed.  Past
        // a list the row is the own one.  (One 2-byte load per iteration,
        // even two iterations ahead, left 0.11 ms of the kernel waiting.)
        const int64_t g0 = goff[blk];
        const int ngb = (int)((goff[blk + 1] - g0) >> 10);      // the block's groups
        const uint64_t *gw = reinterpret_cast<const uint64_t *>(gloc + g0) + threadIdx.x;
        auto word = [&](int gq) __attribute__((always_inline)) {
            return gw[(int64_t)(gq < ngb ? gq : ngb - 1) * 256];
        };
        const int T = (kmax + Q - 1) / Q, ngq = (T + 3) / 4;    // this wave's iterations, groups
        auto four = [&](uint64_t wd, int gq) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (4 * gq + u < T) {                            // wave-uniform
                    const int k = Q * (4 * gq + u) + sub;
                    pair(k < ng ? (int)((wd >> (16 * u)) & 0xffff) : il);
                }
            }
        };
        uint64_t ea = word(0), eb = word(1);
        for (int gq = 0; gq < ngq; gq += 2) {
            const uint64_t wa = ea;
            ea = word(gq + 2);
            four(wa, gq);
            if (gq + 1 >= ngq) break;
            const uint64_t wb = eb;
            eb = word(gq + 3);
            four(wb, gq + 1);
        }
    }
    double sg[G][3];
    quad_scatter<G>(acc, sub, sg);
    if (!active) return;
    // the own state component sub of every group, from the union's row
    double u[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const dvec2 x = ust[il * PU + 2 * g + (sub >> 1)];
        u[g] = (sub & 1) ? x.y : x.x;
    }
    gradient_record_part<G>(sg, u, rec, UD + ic * (16 * G), sub, status);
}

// Transport with the pairs inside a tile evaluated once (FP64, GLF or HLL,
// Hopkins or Ivanova surfaces, G <= 3 groups in one wave: all of them, or one
// of the slices of more, see Slices; two-sided, every pair evaluated by both
// its particles, 4 and 5 groups took 1.13 times as long).  Both solvers' pair
// fluxes and both surfaces are antisymmetric, so one evaluation serves both
// particles of a pair.
//
// A block owns one tile: the 64 consecutive Morton particles of one column
// block of the neighbour table, 16 per wave with 4 lanes each (see below for
// 8).  A particle's task list (k_tasks, built with the geometry) holds its neighbours outside the
// tile and its share of the pairs inside it: an in-tile pair (k, l) is
// evaluated by one of its particles only (chosen to balance the lists'
// lengths), flagged by the sign bit.  That lane adds Phi_kl to its own sum and,
// by an LDS atomic add, to the other particle's row of its own wave's copy of
// the tile's accumulator, which is taken off at the end; the pair's face states
// are the same from either side, so its face-guard counts are taken twice.
// After a block barrier each particle's sum is its own partial sums less the
// waves' rows, in a fixed order, so runs are bitwise reproducible, and the
// in-tile pair flux is antisymmetric bit for bit.  49.5% of the neighbour
// entries of the 128^3 lattice lie inside their tile, so a step evaluates 75%
// of the pair fluxes of a two-sided one.  (With a wave owning a whole tile in 4
// passes the XCD's working set spanned 4 times the particles and its L2 hit
// rate fell from 92% to 38%.)
//
// Q lanes a particle, a tile by Q waves, W waves per SIMD.  Up to 256 tiles
// (one a CU) Q = 8 halves the chain of a particle's pairs: 16^3 particles, 3
// groups, 38.7 -> 33.0 us, 25^3 45.9 -> 36.9; with two tiles a CU it costs
// (32^3 55.2 -> 62.9).  One group of the GLF solver fits W = 3 without much
// spilled (the 32-bit offsets; HLL and more groups do not, the latter for their
// LDS too): from 513 tiles, two a CU, on 48^3 88.5 -> 85.0 us, 100^3 742 ->
// 667; 32^3, where no third one comes, 28.3 -> 30.2.
//
// What bounds it: the load path of the neighbours' rows (texture-data unit busy
// 88% of the time on the 3-group 128^3 lattice and 85% on 926 thousand clustered
// particles; FP64 instructions are half the issue slots; two waves per SIMD wait
// 28% of their cycles).  HLL asks the same path for the table's scattered cells
// (61^3, 2 groups: data 90%, addresses 78% against GLF's 51%).  Guard counts only
// where they are asked for, the partners' sums without a sign change, and the
// shorter reciprocals (rcp64, rsq64) took the lattice from 3.04 to 2.93 ms.  (Rows staged once per tile in LDS, the groups one after the
// other with the pair geometry in registers, cut the rows from L2 sixfold and
// ran 3.33 ms: a fifth more instructions, and barriers between the stages.)
//
// BIN: one tick of the individual-time-step scheme on the tiles.  A pair is
// due when its smaller bin ends a step in this tick, a symmetric condition,
// and its flux weighted by dt 2^min(b_k, b_l) is antisymmetric as before; a
// particle none of whose pairs is due (binm) walks no list.  The particles
// that do not end a step add their sums to the pending sums accm, the others
// apply theirs.
template <int G, bool WHOLE, bool OFF32, bool HLL, bool IVA, bool BIN, int Q, int W>
__global__ __launch_bounds__(64 * Q) __attribute__((amdgpu_waves_per_eu(W, W))) void
k_transport64_tile(int64_t n, int64_t nb, Slices sl, const double *__restrict__ geo,
                   const int32_t *__restrict__ task, const int64_t *__restrict__ wave_base,
                   const int32_t *__restrict__ n_task, const double *__restrict__ UDall,
                   const double *__restrict__ dtp, double c, double box,
                   double *__restrict__ Uout, double *__restrict__ partials,
                   unsigned long long *__restrict__ counts, double *__restrict__ Uung,
                   int32_t *__restrict__ status, const double2 *__restrict__ hll,
                   int64_t tick = 0, double *__restrict__ accm = nullptr,
                   const uint8_t *__restrict__ binm = nullptr) {
    constexpr int NQ = 4 * G, MS = NQ + 1;     // accumulator row, padded against bank conflicts
    static_assert(kTile == 64 && (Q == 4 || Q == 8), "a tile is Q waves of 64 / Q particles");
    constexpr int PW = 64 / Q;                  // particles per wave
    constexpr bool PAD = W == 3;                // rows padded, not swizzled: fewer registers
    __shared__ __attribute__((aligned(16))) double stage[Q][64 * (PAD ? kStage + 1 : kStage)];
    __shared__ double mir[Q][kTile * MS];
    constexpr int DS = 3 * NQ + 1;              // own-gradient row, padded
    __shared__ double dsh[Q][PW * DS];
    __shared__ double smem[Q * 2 * G];
    __shared__ unsigned long long scnt[4];
    // the block's tile and its groups g0 .. g0 + G of the GT
    const int GT = WHOLE ? G : sl.groups, nsl = WHOLE ? 1 : sl.count;
    const int64_t bg = xcd_block(nb * nsl);
    if (bg >= nb * nsl) return;                 // whole block: no barrier is skipped
    const int64_t blk = WHOLE ? bg : bg / nsl;
    const int g0 = WHOLE ? 0 : sl.first + (int)(bg - blk * nsl) * G;
    const double *UD = UDall + 16 * g0;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int sub = lane & (Q - 1);
    const int64_t t0 = blk * kTile;             // the tile's first particle
    const bool wave_live = t0 + PW * wv < n;    // wave-uniform
    const double ibox = 1.0 / box, hc = 0.5 * c, c3 = 3.0 * c;
    if (threadIdx.x < 4) scnt[threadIdx.x] = 0;
    double *sb = stage[wv];
    double *mw = mir[wv];                       // this wave's copy of the accumulator
    for (int e = lane; e < kTile * MS; e += 64) mw[e] = 0.0;
    wave_lds_sync();
    int cE = 0, cF = 0;
    const int pl = PW * wv + lane / Q;       // the lane's particle in the tile
    double acc[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc[q] = 0.0;
    // BIN: this particle ends a step in this tick (ends), or some pair of its
    // neighbourhood is due (touched)
    const int64_t t1 = tick + 1;
    int32_t bk = 0;
    bool ends = true, touched = true;
    if constexpr (BIN) {
        const int64_t icb = t0 + pl < n ? t0 + pl : n - 1;
        bk = (int32_t)geo[(int64_t)kRec * icb + 12];
        const int32_t bm = binm ? (int32_t)binm[icb] : 0;
        ends = (t1 & ((int64_t(1) << bk) - 1)) == 0;
        touched = (t1 & ((int64_t(1) << bm) - 1)) == 0;
    }
    if (wave_live) {
        const int64_t wb = wave_base[blk];
        {
            const int64_t i = t0 + pl;
            const bool active = i < n;
            const int64_t ic = active ? i : n - 1;
            const int32_t nn = (active && touched) ? n_task[i] : 0;
            int32_t kmax = nn;                      // the longest list of the pass
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) kmax = max(kmax, __shfl_xor(kmax, o, 64));
            const double *rk = geo + (int64_t)kRec * ic;
            // IVA: the kernel-gradient sums, slots 13-15 of the records
            const double gk[3] = {IVA ? rk[13] : 0.0, IVA ? rk[14] : 0.0, IVA ? rk[15] : 0.0};
            double Ui[NQ];
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const double *r = UD + (ic * GT + g) * 16;
#pragma unroll
                for (int m = 0; m < 4; ++m) Ui[4 * g + m] = r[m];
            }
            // the own gradients live in LDS (Q lanes read one address); lane
            // sub < 4 copies component sub's
            double *Dsh = dsh[wv] + lane / Q * DS;
            if (Q == 4 || sub < 4) {
#pragma unroll
                for (int g = 0; g < G; ++g)
#pragma unroll
                    for (int a = 0; a < 3; ++a)
                        Dsh[3 * (4 * g + sub) + a] = UD[(ic * GT + g) * 16 + 4 + 3 * sub + a];
            }
            wave_lds_sync();
            const int64_t base = wb + pl;   // the particle's column in the table
            // Lines in flight: v holds the loads of the next stage (the
            // geometry lines, then each group's record lines) while the
            // current stage is evaluated from the stage buffer.  The task of
            // the next iteration is loaded one iteration ahead.
            int32_t tc = sub < nn ? task[base + 64 * (int64_t)sub] : (int32_t)ic;
            int32_t rw[8];
            dvec2 v[8];
            {
                const int32_t j = tc & 0x7fffffff;
#pragma unroll
                for (int m = 0; m < 8; ++m) rw[m] = __shfl(j, 8 * m + (lane >> 3), 64);
                const RowLines<OFF32> gl(geo, rw, 1, lane);
                gl.load(0, v);
            }
            for (int32_t kk = 0; kk < kmax; kk += Q) {
                const int32_t k = kk + sub;
                const bool valid = k < nn;
                const int32_t t = tc;
                // (slot 0 of the tile's table exists once kmax > 0: no branch
                // around the load, whose wait would then be a full one)
                const int32_t tl = task[base + 64 * (int64_t)(k + Q < nn ? k + Q : 0)];
                const int32_t tn = k + Q < nn ? tl : (int32_t)ic;
                const bool mirror = t < 0;
                const int32_t j = t & 0x7fffffff;
                const RowLines<OFF32> ul(UD, rw, GT, lane);
                store_lines<PAD>(v, sb, lane);       // the geometry lines
                ul.load(0, v);
                const Row64<PAD> rl(sb, lane);
                PairGeo pg;
                if constexpr (IVA) {
                    const double gl[3] = {rl[13], rl[14], rl[15]};
                    pair_geometry_ivanova64(rk, rl.f, gk, gl, box, ibox, pg);
                } else {
                    pair_geometry64(rk, rl.f, box, ibox, pg);
                }
                bool use = valid && pg.An > 0.0;
                double wkl = 1.0;                   // BIN: time integration of the exchange
                if constexpr (BIN) {
                    const int32_t bl = (int32_t)rl[12];
                    const int32_t bmin = bk < bl ? bk : bl;
                    use = use && (t1 & ((int64_t(1) << bmin) - 1)) == 0;
                    wkl = ldexp(dtp[0], bmin);
                }
                const double iAn = (HLL && pg.An > 0.0) ? rcp64(pg.An) : 0.0;
                const int cnt2 = mirror ? 2 : 1;
                const int mr = mirror ? (j - (int32_t)t0) * MS : 0;   // the partner's row
#pragma unroll
                for (int g = 0; g < G; ++g) {
                    // the stages in program order: each one's loads stay in
                    // flight across the evaluation of the previous one
                    __builtin_amdgcn_sched_barrier(0);
                    store_lines<PAD>(v, sb, lane);   // group g's record lines
                    if (g + 1 < G) {
                        ul.load(g + 1, v);
                    } else {                    // the next iteration's geometry lines
                        const int32_t jn = tn & 0x7fffffff;
#pragma unroll
                        for (int m = 0; m < 8; ++m) rw[m] = __shfl(jn, 8 * m + (lane >> 3), 64);
                        const RowLines<OFF32> gn(geo, rw, 1, lane);
                        gn.load(0, v);
                    }
                    const Row64<PAD> Rl(sb, lane);
                    double qL[4], qR[4];
#pragma unroll
                    for (int m = 0; m < 4; ++m) {
                        const int q = 4 * g + m;
                        const double dk = Dsh[3 * q] * pg.sx + Dsh[3 * q + 1] * pg.sy + Dsh[3 * q + 2] * pg.sz;
                        const double dl = Rl[4 + 3 * m] * pg.sx + Rl[5 + 3 * m] * pg.sy + Rl[6 + 3 * m] * pg.sz;
                        const double mm = minmod_med(dk, dl);
                        qL[m] = Ui[q] + pg.fk * mm;
                        qR[m] = Rl[m] - pg.fl * mm;
                    }
                    double FAL, aL, bL, FAR, aR, bR;
                    const int f1 = face_m164(qL, pg.Ax, pg.Ay, pg.Az, c, c3, FAL, aL, bL);
                    const int f2 = face_m164(qR, pg.Ax, pg.Ay, pg.Az, c, c3, FAR, aR, bR);
                    double w1 = 0.5, w2 = 0.5, w3 = -hc * pg.An;   // GLF
                    if constexpr (HLL) {
                        double loL, hiL, loR, hiR;
                        hll_speeds64(qL[0], qL[1], qL[2], qL[3], pg.Ax, pg.Ay, pg.Az, iAn, c, hll,
                                     loL, hiL);
                        hll_speeds64(qR[0], qR[1], qR[2], qR[3], pg.Ax, pg.Ay, pg.Az, iAn, c, hll,
                                     loR, hiR);
                        hll_weights(loL, hiL, loR, hiR, pg.An, w1, w2, w3);
                    }
                    if (use) {
                        if (counts) {
                            cE += cnt2 * ((f1 & 1) + (f2 & 1));
                            cF += cnt2 * ((f1 >> 1) + (f2 >> 1));
                        }
                        const double al = __builtin_fma(w1, aL, w2 * aR);
                        const double bl = w1 * bL, br = w2 * bR;
                        double phi[4];
                        phi[0] = __builtin_fma(w3, qR[0] - qL[0], __builtin_fma(w1, FAL, w2 * FAR));
                        const double Av[3] = {pg.Ax, pg.Ay, pg.Az};
#pragma unroll
                        for (int m = 1; m < 4; ++m)
                            phi[m] = __builtin_fma(w3, qR[m] - qL[m],
                                                   __builtin_fma(al, Av[m - 1],
                                                                 __builtin_fma(bl, qL[m], br * qR[m])));
                        if constexpr (BIN) {
#pragma unroll
                            for (int m = 0; m < 4; ++m) phi[m] *= wkl;
                        }
#pragma unroll
                        for (int m = 0; m < 4; ++m) acc[4 * g + m] += phi[m];
                        if (mirror) {
#pragma unroll
                            for (int m = 0; m < 4; ++m) atomicAdd(mw + mr + 4 * g + m, phi[m]);
                        }
                    }
                }
                tc = tn;
                __builtin_amdgcn_sched_barrier(0);
            }
            // the Q lanes' partial sums, combined by a fixed butterfly
#pragma unroll
            for (int q = 0; q < NQ; ++q) {
                quad_sum<4>(acc[q]);
                if constexpr (Q == 8) acc[q] += __shfl_xor(acc[q], 4, 64);
            }
        }
    }
    // every wave's deposits are in its copy of the accumulator
    __syncthreads();
    // update, post-update guard, ledger, photon budget: the first lane of each
    // particle; its sum is its own partial sums less the waves' rows, in
    // that fixed order
    const int64_t i = t0 + pl;
    const bool owner = wave_live && sub == 0 && i < n;
    double red[2 * G];
    int gE = 0, gF = 0;
    double chk = 0.0;   // NaN iff an updated state is NaN or infinite
    if (BIN && owner && !ends) {
        // no update in this tick: keep the pending sums, count the current state
        const double V = geo[(int64_t)kRec * i + R_V];
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int v = 0; v < Q; ++v) acc[q] -= mir[v][pl * MS + q];
#pragma unroll
        for (int g = 0; g < G; ++g) {
            if (touched) {
                double *a = accm + (i * GT + g0 + g) * 4;
#pragma unroll
                for (int m = 0; m < 4; ++m) a[m] += acc[4 * g + m];
            }
            red[g] = V * UD[(i * GT + g) * 16];
            red[G + g] = 0.0;
        }
    } else if (owner) {
        const double V = geo[(int64_t)kRec * i + R_V];
        // the update: U - dt/V sum (global step), or U - (pending + this tick)/V
        const double dtV = BIN ? 1.0 / V : dtp[0] / V;
#pragma unroll
        for (int q = 0; q < NQ; ++q)
#pragma unroll
            for (int v = 0; v < Q; ++v) acc[q] -= mir[v][pl * MS + q];
        if constexpr (BIN) {
#pragma unroll
            for (int g = 0; g < G; ++g) {
                double *a = accm + (i * GT + g0 + g) * 4;
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    acc[4 * g + m] += a[m];
                    a[m] = 0.0;
                }
            }
        }
#pragma unroll
        for (int g = 0; g < G; ++g) {
            const double *u = UD + (i * GT + g) * 16;
            double q0 = u[0] - dtV * acc[4 * g + 0];
            double q1 = u[1] - dtV * acc[4 * g + 1];
            double q2 = u[2] - dtV * acc[4 * g + 2];
            double q3 = u[3] - dtV * acc[4 * g + 3];
            const double Epre = q0;
            chk = __builtin_fma(q0, 0.0, chk);
            chk = __builtin_fma(q1, 0.0, chk);
            chk = __builtin_fma(q2, 0.0, chk);
            chk = __builtin_fma(q3, 0.0, chk);
            if (Uung) {
                double *uu = Uung + (i * GT + g0 + g) * 4;
                uu[0] = q0;
                uu[1] = q1;
                uu[2] = q2;
                uu[3] = q3;
            }
            const int f = guard64(q0, q1, q2, q3, c);
            gE += f & 1;
            gF += f >> 1;
            double *o = Uout + (i * GT + g0 + g) * 4;
            o[0] = q0;
            o[1] = q1;
            o[2] = q2;
            o[3] = q3;
            red[g] = V * q0;
            red[G + g] = (f & 1) ? -Epre * V : 0.0;
        }
    } else {
#pragma unroll
        for (int p = 0; p < 2 * G; ++p) red[p] = 0.0;
    }
    if (chk != chk) atomicOr(status, ST_NONFINITE);
    if (partials)
        block_reduce_store<2 * G, Q>(red, partials + blk * 2 * GT, smem,
                                  [&](int p) { return p < G ? g0 + p : GT + g0 + p - G; });
    if (counts) {
        int64_t v0 = wave_sum_i64(cE), v1 = wave_sum_i64(cF), v2 = wave_sum_i64(gE),
                v3 = wave_sum_i64(gF);
        __syncthreads();
        if ((threadIdx.x & 63) == 0) {
            atomicAdd(&scnt[0], (unsigned long long)v0);
            atomicAdd(&scnt[1], (unsigned long long)v1);
            atomicAdd(&scnt[2], (unsigned long long)v2);
            atomicAdd(&scnt[3], (unsigned long long)v3);
        }
        __syncthreads();
        if (threadIdx.x < 4 && scnt[threadIdx.x]) atomicAdd(&counts[threadIdx.x], scnt[threadIdx.x]);
    }
}

// ---------------------------------------------------------------------------
// Photon budget Q_g = sum_k V_k E_kg: block partials, then one block combines
// them with compensated (two-sum) arithmetic in a fixed order.
template <typename T>
__global__ __launch_bounds__(kBlock) void k_total_partials(int64_t n, int G,
                                                           const double *__restrict__ geo,
                                                           const T *__restrict__ U,
                                                           double *__restrict__ partials) {
    __shared__ double smem[kBlock];
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    for (int g = 0; g < G; ++g) {
        double v = (i < n) ? geo[(int64_t)kRec * i + R_V] * (double)U[(i * G + g) * 4] : 0.0;
        smem[threadIdx.x] = v;
        __syncthreads();
        for (int s = kBlock / 2; s > 0; s >>= 1) {
            if (threadIdx.x < s) smem[threadIdx.x] += smem[threadIdx.x + s];
            __syncthreads();
        }
        if (threadIdx.x == 0) partials[(int64_t)blockIdx.x * 2 * G + g] = smem[0];
        __syncthreads();
    }
}

__device__ __forceinline__ void two_sum(double a, double b, double &s, double &e) {
    s = a + b;
    double bb = s - a;
    e = (a - (s - bb)) + (b - bb);
}

// part [nb][2G]: columns 0..G-1 photon totals, G..2G-1 ledger.  Q[g] = sum (written),
// ledger[g] += sum, in a fixed order: thread t of a block sums whole rows t,
// t + kBlock, ... of the block's share (consecutive threads read consecutive
// rows), one compensated sum per column; the threads' sums of all columns meet
// in a fixed tree, over the lanes by shuffles, then over the waves.  Up to
// kFinOneRows rows are one block's work; more are kFinBlocks blocks' and
// their compensated sums a second launch's.  (Two launches whatever the rows,
// and a tree through LDS per column, were 7.8 of the 32 us of a step of 16^3
// particles.)
constexpr int kFinBlocks = 32;
constexpr int64_t kFinOneRows = 2048;

// The compensated pairs (s, e) of the block's W waves, summed, in lane 0 of wave 0.
template <int C, int W>
__device__ __forceinline__ void block_two_sum(double (&s)[C], double (&e)[C],
                                              double (&sh)[W][C][2]) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    auto add = [](double &s0, double &e0, double s1, double e1) {
        double t, err;
        two_sum(s0, s1, t, err);
        s0 = t;
        e0 += e1 + err;
    };
#pragma unroll
    for (int o = 32; o > 0; o >>= 1)
#pragma unroll
        for (int c = 0; c < C; ++c)
            add(s[c], e[c], __shfl_down(s[c], o, 64), __shfl_down(e[c], o, 64));
    if constexpr (W > 1) {
        if (lane == 0) {
#pragma unroll
            for (int c = 0; c < C; ++c) {
                sh[wv][c][0] = s[c];
                sh[wv][c][1] = e[c];
            }
        }
        __syncthreads();
        if (threadIdx.x == 0) {
#pragma unroll
            for (int c = 0; c < C; ++c)
                for (int w = 1; w < W; ++w) add(s[c], e[c], sh[w][c][0], sh[w][c][1]);
        }
    }
}

template <int C>
__device__ __forceinline__ void sum_rows(int64_t r0, int64_t r1, const double *__restrict__ part,
                                         double (&s)[C], double (&e)[C]) {
#pragma unroll
    for (int c = 0; c < C; ++c) s[c] = e[c] = 0.0;
    for (int64_t b = r0 + threadIdx.x; b < r1; b += kBlock) {
        const double *row = part + b * C;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            double t, err;
            two_sum(s[c], row[c], t, err);
            s[c] = t;
            e[c] += err;
        }
    }
}

template <int G>
__device__ __forceinline__ void store_totals(const double (&s)[2 * G], const double (&e)[2 * G],
                                             double *__restrict__ Q, double *__restrict__ ledger) {
#pragma unroll
    for (int g = 0; g < G; ++g) {
        if (Q) Q[g] = s[g] + e[g];
        if (ledger) ledger[g] += s[G + g] + e[G + g];
    }
}

template <int G>
__global__ __launch_bounds__(kBlock) void k_finalize_one(int64_t nb, const double *__restrict__ part,
                                                         double *__restrict__ Q,
                                                         double *__restrict__ ledger) {
    __shared__ double sh[kBlock / 64][2 * G][2];
    double s[2 * G], e[2 * G];
    sum_rows<2 * G>(0, nb, part, s, e);
    block_two_sum<2 * G, kBlock / 64>(s, e, sh);
    if (threadIdx.x == 0) store_totals<G>(s, e, Q, ledger);
}

template <int G>
__global__ __launch_bounds__(kBlock) void k_finalize_rows(int64_t nb, const double *__restrict__ part,
                                                          double *__restrict__ fin) {
    constexpr int C = 2 * G;
    __shared__ double sh[kBlock / 64][C][2];
    const int64_t m = (nb + kFinBlocks - 1) / kFinBlocks;
    const int64_t r0 = blockIdx.x * m;
    double s[C], e[C];
    sum_rows<C>(r0, min(nb, r0 + m), part, s, e);
    block_two_sum<C, kBlock / 64>(s, e, sh);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int c = 0; c < C; ++c) {
            fin[(blockIdx.x * C + c) * 2] = s[c];
            fin[(blockIdx.x * C + c) * 2 + 1] = e[c];
        }
    }
}

template <int G>
__global__ __launch_bounds__(64) void k_finalize(const double *__restrict__ fin,
                                                 double *__restrict__ Q,
                                                 double *__restrict__ ledger) {
    constexpr int C = 2 * G;
    __shared__ double sh[1][C][2];
    double s[C], e[C];
    const bool in = threadIdx.x < kFinBlocks;
#pragma unroll
    for (int c = 0; c < C; ++c) {
        s[c] = in ? fin[(threadIdx.x * C + c) * 2] : 0.0;
        e[c] = in ? fin[(threadIdx.x * C + c) * 2 + 1] : 0.0;
    }
    block_two_sum<C, 1>(s, e, sh);
    if (threadIdx.x == 0) store_totals<G>(s, e, Q, ledger);
}

// part is ctx->partials; the kFinBlocks x 2G compensated pairs of a first pass
// go to the slack the buffer keeps after its rows.
template <int G>
void launch_finalize(rt_ctx *ctx, int64_t nb, const double *part, double *Q, double *ledger) {
    if (nb <= kFinOneRows) {
        k_finalize_one<G><<<1, kBlock, 0, ctx->stream>>>(nb, part, Q, ledger);
        return;
    }
    double *fin = ctx->partials + 2 * G * ctx->nblocks;
    k_finalize_rows<G><<<kFinBlocks, kBlock, 0, ctx->stream>>>(nb, part, fin);
    k_finalize<G><<<1, 64, 0, ctx->stream>>>(fin, Q, ledger);
}

// rows of block partials the FP64 transport writes (one per tile)
inline int64_t transport64_rows(int64_t n) { return (n + kTile - 1) / kTile; }

constexpr int64_t kWideTiles = 256, kThreeTiles = 512;
// The tile transport of G groups of all GT, or of slices of G of them; accm: one
// tick of the individual time steps.
template <int G, bool WHOLE>
void launch_tiles64(rt_ctx *ctx, Slices sl, const double *UD, const double *dt, double *Uout,
                    double *partials, int64_t *counts, double *Uung, int64_t tick, double *accm) {
    const int64_t n = ctx->p.n, nt = transport64_rows(n);
    const bool hll = ctx->solver == RT_HLL, iva = ctx->surfaces == RT_IVANOVA;
    // rows addressed by 32-bit offsets while the gradient records fit 4 GiB
    const bool off32 = (uint64_t)n * 128u * ctx->p.groups < (uint64_t(1) << 32);
    const int64_t blocks = nt * (WHOLE ? 1 : sl.count);
    const unsigned grid = (unsigned)xcd_grid(blocks);
    // lanes per particle and waves per SIMD: see k_transport64_tile
    const bool wide = blocks <= kWideTiles, three = blocks > kThreeTiles;
    if (wide && off32) rt_route(ctx, "wide");
    if (three && G == 1 && off32 && !hll) rt_route(ctx, "three_waves");
    // (one group a block is for few blocks, so its records are far below 4 GiB,
    // and two groups in a wave for more than 256)
    constexpr bool ALL32 = G == 1 && !WHOLE, WIDE = !(G == 2 && WHOLE);
#define RT_TILE_LAUNCH_QW(OFF32_, HLL_, IVA_, BIN_, Q_, W_)                                      \
    k_transport64_tile<G, WHOLE, OFF32_, HLL_, IVA_, BIN_, Q_, W_>                               \
        <<<grid, 64 * Q_, 0, ctx->stream>>>(                                                     \
        n, nt, sl, ctx->geo, ctx->task, ctx->wave_base, ctx->n_task, UD, dt, ctx->p.c_red,       \
        ctx->p.box, Uout, partials, (unsigned long long *)counts, Uung, ctx->status,             \
        (const double2 *)ctx->hll_table, tick, accm, ctx->bin8 ? ctx->bin8 + n : nullptr)
#define RT_TILE_LAUNCH(OFF32_, HLL_, IVA_, BIN_)                                                 \
    do {                                                                                         \
        if constexpr (OFF32_ && WIDE) {                                                          \
            if (wide) {                                                                          \
                RT_TILE_LAUNCH_QW(OFF32_, HLL_, IVA_, BIN_, 8, 2);                               \
                break;                                                                           \
            }                                                                                    \
        }                                                                                        \
        if constexpr (G == 1 && OFF32_ && !HLL_) {                                               \
            if (three) {                                                                         \
                RT_TILE_LAUNCH_QW(OFF32_, HLL_, IVA_, BIN_, 4, 3);                               \
                break;                                                                           \
            }                                                                                    \
        }                                                                                        \
        RT_TILE_LAUNCH_QW(OFF32_, HLL_, IVA_, BIN_, 4, 2);                                       \
    } while (0)
#define RT_TILE_LAUNCH_B(OFF32_, HLL_, IVA_)                                                     \
    do {                                                                                         \
        if (accm) {                                                                              \
            RT_TILE_LAUNCH(OFF32_, HLL_, IVA_, true);                                            \
        } else {                                                                                 \
            RT_TILE_LAUNCH(OFF32_, HLL_, IVA_, false);                                           \
        }                                                                                        \
    } while (0)
#define RT_TILE_LAUNCH_S(HLL_, IVA_)                                                             \
    do {                                                                                         \
        if (ALL32 || off32) RT_TILE_LAUNCH_B(true, HLL_, IVA_);                                  \
        else RT_TILE_LAUNCH_B(ALL32, HLL_, IVA_);                                                \
    } while (0)
    if (hll && iva) RT_TILE_LAUNCH_S(true, true);
    else if (hll) RT_TILE_LAUNCH_S(true, false);
    else if (iva) RT_TILE_LAUNCH_S(false, true);
    else RT_TILE_LAUNCH_S(false, false);
#undef RT_TILE_LAUNCH_S
#undef RT_TILE_LAUNCH_B
#undef RT_TILE_LAUNCH
#undef RT_TILE_LAUNCH_QW
}

void launch_transport64(rt_ctx *ctx, const double *UD, const double *dt, double *Uout,
                        double *partials, int64_t *counts, double *Uung, int64_t tick,
                        double *accm) {
    const int G = ctx->p.groups, s3 = slices_of_3(G), s2 = slices_of_2(G);
    const Slices sl{G, 0, s3};
    const bool few = G > 1 && transport64_rows(ctx->p.n) * G <= one_group_blocks(true, G);
    rt_route(ctx, few ? "one_group" : G <= 3 ? "whole" : "slices");
    if (few) {
        launch_tiles64<1, false>(ctx, Slices{G, 0, G}, UD, dt, Uout, partials, counts, Uung, tick,
                                 accm);
    } else if (G == 1) {
        launch_tiles64<1, true>(ctx, sl, UD, dt, Uout, partials, counts, Uung, tick, accm);
    } else if (G == 2) {
        launch_tiles64<2, true>(ctx, sl, UD, dt, Uout, partials, counts, Uung, tick, accm);
    } else if (G == 3) {
        launch_tiles64<3, true>(ctx, sl, UD, dt, Uout, partials, counts, Uung, tick, accm);
    } else {
        if (s3 > 0)
            launch_tiles64<3, false>(ctx, sl, UD, dt, Uout, partials, counts, Uung, tick, accm);
        if (s2 > 0)
            launch_tiles64<2, false>(ctx, Slices{G, 3 * s3, s2}, UD, dt, Uout, partials, counts,
                                     Uung, tick, accm);
    }
}

// The ticks' gradients from the neighbour unions; 0: staged.
#ifndef RT_TICK_UNION
#define RT_TICK_UNION 1
#endif

// Lanes per particle of the FP64 gradient (1, 2 or 4); Q = 4 measured 14%
// faster than Q = 1 on the 3-group 128^3 lattice.
#ifndef RT_GRADIENT_Q
#define RT_GRADIENT_Q 4
#endif
constexpr int kGQ = RT_GRADIENT_Q;

template <int G>
void launch_gradient64(rt_ctx *ctx, const double *U, double *UD) {
    constexpr int B = grad_block(G);
    if constexpr (union_cap(G) > 0 && kGQ == 4 && B == 256) {
        if (ctx->urows) {
            // blocks whose union fits: from LDS; a few larger ones: too, one to a
            // CU; the others: staged, by list
            const int64_t nw = ctx->nwaves;
#define RT_UNION_LAUNCH(W_)                                                                    \
    k_gradient64u<G, kGQ, W_><<<(unsigned)xcd_grid(nw), kBlock, 0, ctx->stream>>>(            \
        ctx->p.n, nw, ctx->geo, ctx->xs, ctx->urow, ctx->urows, ctx->gloc, ctx->goff,          \
        ctx->uown, ctx->n_gath, U, UD, ctx->status, ctx->p.box)
            if constexpr (union_cap3(G) > 0) {
                if (ctx->union_waves == 3) RT_UNION_LAUNCH(3);
                else RT_UNION_LAUNCH(2);
            } else {
                RT_UNION_LAUNCH(2);
            }
#undef RT_UNION_LAUNCH
            if constexpr (union_cap_large(G) > 0) {
                if (ctx->n_lblk > 0) rt_route(ctx, "large");
                if (ctx->n_lblk > 0)
                    k_gradient64u<G, kGQ, 1><<<(unsigned)xcd_grid(ctx->n_lblk), kBlock, 0,
                                               ctx->stream>>>(
                        ctx->p.n, ctx->n_lblk, ctx->geo, ctx->xs, ctx->lrow, ctx->lrows, ctx->gloc,
                        ctx->goff, ctx->uown, ctx->n_gath, U, UD, ctx->status, ctx->p.box, 0,
                        ctx->ublk + 2);
            }
            if (ctx->n_sblk > 0) rt_route(ctx, "staged");
            if (ctx->n_sblk > 0)
                k_gradient64<G, false, kGQ><<<(unsigned)xcd_grid(ctx->n_sblk), B, 0, ctx->stream>>>(
                    ctx->p.n, ctx->n_sblk, ctx->geo, ctx->xs, ctx->nbr, ctx->wave_base, ctx->n_gath,
                    U, UD, ctx->status, ctx->p.box, 0, ctx->sblk);
            return;
        }
    }
    const int64_t n = ctx->p.n, nb = (n + B / kGQ - 1) / (B / kGQ);
    k_gradient64<G, false, kGQ><<<(unsigned)xcd_grid(nb), B, 0, ctx->stream>>>(
        n, nb, ctx->geo, ctx->xs, ctx->nbr, ctx->wave_base, ctx->n_gath, U, UD, ctx->status,
        ctx->p.box);
}

template <int G>
void launch_tick64(rt_ctx *ctx, const double *U, double *UD, const double *dt, double *Uout,
                   double *partials, int64_t *counts, int64_t tick, double *accm) {
    const int64_t n = ctx->p.n;
    constexpr int B = grad_block(G);
    const int64_t ng = (n + B / kGQ - 1) / (B / kGQ);
    bool grad_done = false;
    if constexpr (union_cap(G) > 0 && kGQ == 4 && B == 256) {
        if (RT_TICK_UNION != 0 && ctx->urows) {
            // the neighbour unions, in their time-bin mode; the blocks whose
            // union does not fit: staged, by list
            const int64_t nw = ctx->nwaves;
#define RT_TICK_UNION_LAUNCH(W_)                                                               \
    k_gradient64u<G, kGQ, W_, true><<<(unsigned)xcd_grid(nw), kBlock, 0, ctx->stream>>>(      \
        n, nw, ctx->geo, ctx->xs, ctx->urow, ctx->urows, ctx->gloc, ctx->goff, ctx->uown,       \
        ctx->n_gath, U, UD, ctx->status, ctx->p.box, tick)
            if constexpr (union_cap3(G) > 0) {
                if (ctx->union_waves == 3) RT_TICK_UNION_LAUNCH(3);
                else RT_TICK_UNION_LAUNCH(2);
            } else {
                RT_TICK_UNION_LAUNCH(2);
            }
#undef RT_TICK_UNION_LAUNCH
            if constexpr (union_cap_large(G) > 0) {
                if (ctx->n_lblk > 0) rt_route(ctx, "large");
                if (ctx->n_lblk > 0)
                    k_gradient64u<G, kGQ, 1, true><<<(unsigned)xcd_grid(ctx->n_lblk), kBlock, 0,
                                                     ctx->stream>>>(
                        n, ctx->n_lblk, ctx->geo, ctx->xs, ctx->lrow, ctx->lrows, ctx->gloc,
                        ctx->goff, ctx->uown, ctx->n_gath, U, UD, ctx->status, ctx->p.box, tick,
                        ctx->ublk + 2);
            }
            if (ctx->n_sblk > 0) rt_route(ctx, "staged");
            if (ctx->n_sblk > 0)
                k_gradient64<G, true, kGQ><<<(unsigned)xcd_grid(ctx->n_sblk), B, 0, ctx->stream>>>(
                    n, ctx->n_sblk, ctx->geo, ctx->xs, ctx->nbr, ctx->wave_base, ctx->n_gath,
                    U, UD, ctx->status, ctx->p.box, tick, ctx->sblk);
            grad_done = true;
        }
    }
    if (!grad_done)
        k_gradient64<G, true, kGQ><<<(unsigned)xcd_grid(ng), B, 0, ctx->stream>>>(
            n, ng, ctx->geo, ctx->xs, ctx->nbr, ctx->wave_base, ctx->n_gath, U, UD, ctx->status,
            ctx->p.box, tick);
    launch_transport64(ctx, UD, dt, Uout, partials, counts, nullptr, tick, accm);
}

#define RT_DISPATCH_G(G_, FN, ...)                                  \
    switch (G_) {                                                   \
        case 1: FN<1>(__VA_ARGS__); break;                          \
        case 2: FN<2>(__VA_ARGS__); break;                          \
        case 3: FN<3>(__VA_ARGS__); break;                          \
        case 4: FN<4>(__VA_ARGS__); break;                          \
        case 5: FN<5>(__VA_ARGS__); break;                          \
        case 6: FN<6>(__VA_ARGS__); break;                          \
        case 7: FN<7>(__VA_ARGS__); break;                          \
        case 8: FN<8>(__VA_ARGS__); break;                          \
        default: break;                                             \
    }

}  // namespace

// Combine nb rows of ctx->partials into Q (columns 0..G-1, written) and
// ledger (columns G..2G-1, accumulated); either may be NULL.
void rt_finalize_partials(rt_ctx *ctx, int64_t nb, double *Q, double *ledger) {
    RT_DISPATCH_G(ctx->p.groups, launch_finalize, ctx, nb, ctx->partials, Q, ledger);
}

rt_status rt_ensure_partials(rt_ctx *ctx) {
    // enough rows for every kernel that writes them: one per tile at most
    const int64_t nb = transport64_rows(ctx->p.n);
    if (ctx->partials && ctx->nblocks >= nb) return RT_OK;
    rt_free(ctx, ctx->partials);
    ctx->partials = nullptr;
    // the rows, then the first pass of the finalize (kFinBlocks x 2G pairs)
    rt_status rs = rt_alloc(ctx, (void **)&ctx->partials,
                            sizeof(double) * 2 * ctx->p.groups * (nb + 2 * kFinBlocks));
    if (rs != RT_OK) return rs;
    ctx->nblocks = nb;
    return RT_OK;
}

rt_status rt_inject_impl(rt_ctx *ctx, void *U, const double *L, const double *dt) {
    if (ctx->S == 0 || ctx->n_inj_gas == 0) return RT_OK;
    rt_timer_begin(ctx, "inject");
    if (ctx->p.precision == RT_FP64)
        k_inject<double><<<nblk(ctx->n_inj_gas), kBlock, 0, ctx->stream>>>(
            ctx->n_inj_gas, ctx->p.groups, ctx->inj_gptr, ctx->inj_gas, ctx->inj_src,
            ctx->inj_coef, L, dt, (double *)U);
    else
        k_inject<float><<<nblk(ctx->n_inj_gas), kBlock, 0, ctx->stream>>>(
            ctx->n_inj_gas, ctx->p.groups, ctx->inj_gptr, ctx->inj_gas, ctx->inj_src,
            ctx->inj_coef, L, dt, (float *)U);
    rt_timer_end(ctx, "inject");
    RT_HIP(hipGetLastError());
    return RT_OK;
}

rt_status rt_gradient_impl(rt_ctx *ctx, const void *U, void *UD) {
    rt_timer_begin(ctx, "gradient");
    if (ctx->p.precision == RT_FP64) {
        RT_DISPATCH_G(ctx->p.groups, launch_gradient64, ctx, (const double *)U, (double *)UD);
    } else {
        rt_gradient32(ctx, (const float *)U, (float *)UD);
    }
    rt_timer_end(ctx, "gradient");
    RT_HIP(hipGetLastError());
    return RT_OK;
}

rt_status rt_transport_impl(rt_ctx *ctx, const void *UD, const double *dt, void *U_out,
                            double *Q, int64_t *counts, double *ledger, void *Uung) {
    // rows of block partials: the FP64 kernel's blocks, or one per kBlock particles
    const int64_t nb = ctx->p.precision == RT_FP64 ? transport64_rows(ctx->p.n)
                                                   : rt_transport32_rows(ctx->p.n);
    double *part = (Q || ledger) ? ctx->partials : nullptr;
    rt_timer_begin(ctx, "transport");
    if (ctx->p.precision == RT_FP64) {
        launch_transport64(ctx, (const double *)UD, dt, (double *)U_out, part, counts,
                           (double *)Uung, 0, nullptr);
    } else {
        rt_transport32(ctx, (const float *)UD, dt, (float *)U_out, part, counts, (float *)Uung);
    }
    rt_timer_end(ctx, "transport");
    RT_HIP(hipGetLastError());
    if (part) {
        RT_DISPATCH_G(ctx->p.groups, launch_finalize, ctx, nb, part, Q, ledger);
        RT_HIP(hipGetLastError());
    }
    return RT_OK;
}

// Gradient and transport of one tick of the individual-time-step scheme
// (FP64; injection and the refresh of the stored states are in rt_bins.hip).
rt_status rt_tick_step_impl(rt_ctx *ctx, double *U, double *UD, const double *dt, int64_t tick,
                            double *accm, double *Q, int64_t *counts, double *ledger) {
    const int64_t nb = transport64_rows(ctx->p.n);
    double *part = (Q || ledger) ? ctx->partials : nullptr;
    rt_timer_begin(ctx, "tick");
    RT_DISPATCH_G(ctx->p.groups, launch_tick64, ctx, U, UD, dt, U, part, counts, tick, accm);
    rt_timer_end(ctx, "tick");
    RT_HIP(hipGetLastError());
    if (part) {
        RT_DISPATCH_G(ctx->p.groups, launch_finalize, ctx, nb, part, Q, ledger);
        RT_HIP(hipGetLastError());
    }
    return RT_OK;
}

rt_status rt_total_impl(rt_ctx *ctx, const void *U, double *Q) {
    const int64_t n = ctx->p.n, nb = (n + kBlock - 1) / kBlock;
    if (ctx->p.precision == RT_FP64)
        k_total_partials<double><<<(unsigned)nb, kBlock, 0, ctx->stream>>>(
            n, ctx->p.groups, ctx->geo, (const double *)U, ctx->partials);
    else
        k_total_partials<float><<<(unsigned)nb, kBlock, 0, ctx->stream>>>(
            n, ctx->p.groups, ctx->geo, (const float *)U, ctx->partials);
    RT_DISPATCH_G(ctx->p.groups, launch_finalize, ctx, nb, ctx->partials, Q, nullptr);
    RT_HIP(hipGetLastError());
    return RT_OK;
}
