// Compensated-FP32 adjoint of one RT step: the passes of the FP64 adjoint
// (guard VJP, pair VJPs, transpose of the gradient) with FP32 pair
// arithmetic; the state cotangent of every particle is summed with Kahan
// compensation.
#include "rt_pair32.h"

using namespace gearrt;

namespace {

inline unsigned nblk(int64_t n, int b = kBlock) { return (unsigned)((n + b - 1) / b); }

template <int G>
__global__ __launch_bounds__(kBlock) void k_adj_guard32(int64_t n, const float *__restrict__ Uung,
                                                        const float *__restrict__ lam_next,
                                                        float *__restrict__ lam2, float c) {
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n * G) return;
    float q[4], l[4];
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        q[m] = Uung[4 * t + m];
        l[m] = lam_next[4 * t + m];
    }
    guard32_vjp(q, l, c);
#pragma unroll
    for (int m = 0; m < 4; ++m) lam2[4 * t + m] = l[m];
}

// Exchange among the 4 lanes of a quad: v[u] of lane m becomes v[m] of lane u.
__device__ __forceinline__ void quad_transpose(float (&v)[4], int sub) {
    // (values, not elements, in the conditions: a chosen element would put the
    // array into memory)
    const bool o1 = sub & 1, o2 = sub & 2;
#pragma unroll
    for (int r = 0; r < 4; r += 2) {
        const float a = v[r], b = v[r + 1];
        const float t = quad_xor<1>(o1 ? +a : +b);
        v[r] = o1 ? +t : +a;
        v[r + 1] = o1 ? +b : +t;
    }
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const float a = v[r], b = v[r + 2];
        const float t = quad_xor<2>(o2 ? +a : +b);
        v[r] = o2 ? +t : +a;
        v[r + 2] = o2 ? +b : +t;
    }
}

// Pass B (as in the FP64 adjoint; every pair from both its particles), one
// group a block.  A quad of lanes shares a particle: each pulls back every
// fourth of its pairs, then the quad exchanges the four pairs' cotangents and
// lane m sums component m (its state cotangent compensated) over all of them in
// list order, with the operations of one lane per particle, so with the same
// bits.  With one lane per particle a wave reached 64 neighbourhoods, one row
// after the other, and waited for memory: 377 us for 4 groups of 58 thousand
// clustered particles, now 262; the 100^3 lattice, 3 groups, is bound by its
// vector instructions (whole backward step 2.94 -> 2.82 ms, HLL 4.65 -> 4.44).
// The geometry rows are in flight one iteration ahead, a group's rows across
// the pair geometry.  (On the tiles, pairs inside evaluated once, the FP32 sums,
// and with them dL, round differently, and it was no faster: 300 us.)
// HLL and IVA as in the FP64 pass (the FP32 table, the FP32 Ivanova surfaces of
// the FP32C transport).
template <bool OFF32, bool HLL, bool IVA>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(3))) void
k_adj_pair32(int64_t n, int64_t nb, int G, const float *__restrict__ geo32,
                  const double *__restrict__ geo, const int32_t *__restrict__ nbr,
                  const int64_t *__restrict__ wave_base, const int32_t *__restrict__ n_nbr,
                  const float *__restrict__ UD, const float *__restrict__ lam2,
                  const double *__restrict__ dtp, double c, double box, float *__restrict__ R,
                  const float2 *__restrict__ hll, const double *__restrict__ ivan) {
    static_assert(kBlock == 256, "a block of 4 waves x 16 particles per column block");
    __shared__ __attribute__((aligned(16))) float stage[kBlock / 64][64 * kStage32];
    const int64_t bg = xcd_block(nb * G);
    if (bg >= nb * G) return;
    const int64_t blk = bg / G;
    const int g0 = (int)(bg - blk * G);
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int sub = lane & 3;
    const int pl = 16 * wv + (lane >> 2);       // the lane's particle in the column block
    const int64_t i = blk * 64 + pl;
    const bool active = i < n;
    const int64_t ic = active ? i : n - 1;
    const bool wave_live = blk * 64 + 16 * wv < n;   // wave-uniform
    const double ibox = 1.0 / box;
    const float cf = (float)c, c2 = (float)(c * c), ic2 = (float)(1.0 / (c * c));
    const float dtf = (float)dtp[0];
    float *sb = stage[wv];

    const float *rk = geo32 + (int64_t)F_REC * ic;
    const double *xk = reinterpret_cast<const double *>(rk);
    const double pkx = xk[0], pky = xk[1], pkz = xk[2];
    const float iHk = rk[F_IH], hk = rk[F_H];
    float gk[3] = {0.0f, 0.0f, 0.0f};   // IVA: own kernel-gradient sum
    if (IVA) {
        gk[0] = (float)ivan[4 * ic];
        gk[1] = (float)ivan[4 * ic + 1];
        gk[2] = (float)ivan[4 * ic + 2];
    }
    float Bk[6];
#pragma unroll
    for (int a = 0; a < 6; ++a) Bk[a] = rk[F_B + a];
    const float dtVk = (float)(dtp[0] / geo[(int64_t)kRec * ic + R_V]);
    float Ui[4], Di[12], Li[4];
    const float *ro = UD + (ic * G + g0) * 16;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        Ui[m] = ro[m];
        Di[3 * m + 0] = ro[4 + 3 * m];
        Di[3 * m + 1] = ro[5 + 3 * m];
        Di[3 * m + 2] = ro[6 + 3 * m];
        Li[m] = lam2[(ic * G + g0) * 4 + m];
    }
    // component sub's sums
    Kahan aU{0.0f, 0.0f};
    float aD[3] = {0.0f, 0.0f, 0.0f};
    if (wave_live) {
        const int64_t base = wave_base[blk] + pl;   // the particle's column in the table
        const int32_t nn = active ? n_nbr[i] : 0;
        int32_t kmax = nn;                          // the longest list of the wave
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) kmax = max(kmax, __shfl_xor(kmax, o, 64));
        // the next iteration's neighbour, and its geometry row, are in flight
        // while this one is evaluated
        int32_t jn = sub < nn ? nbr[base + 64 * (int64_t)sub] : (int32_t)ic;
        uint32_t row[4];
        fvec4 v[4];
        {
#pragma unroll
            for (int m = 0; m < 4; ++m) row[m] = __shfl(jn, 16 * m + (lane >> 2), 64);
            load_rows32<OFF32>(geo32, row, lane, v);
        }
        for (int32_t kk = 0; kk < kmax; kk += 4) {
            const int32_t k = kk + sub;
            const bool valid = k < nn;
            const int32_t j = jn;
            // (slot 0 of the block's table exists once kmax > 0: no branch
            // around the load, whose wait would then be a full one)
            const int32_t jl = nbr[base + 64 * (int64_t)(k + 4 < nn ? k + 4 : 0)];
            jn = k + 4 < nn ? jl : (int32_t)ic;
            store_rows32(v, sb, lane);          // the geometry rows
            // the group's record rows and cotangents in one round trip
            {
                uint32_t rowg[4];
#pragma unroll
                for (int m = 0; m < 4; ++m) rowg[m] = row[m] * G + g0;
                load_rows32<OFF32>(UD, rowg, lane, v);
            }
            const fvec4 Ll = *reinterpret_cast<const fvec4 *>(lam2 + ((int64_t)j * G + g0) * 4);
            PairGeo32 pg;
            const Row32 rl(sb, lane);
            pair_geometry32(pkx, pky, pkz, iHk, hk, Bk, rl, box, ibox, pg);
            if (IVA) {                          // the same pair with the Ivanova surface
                const double *gd = ivan + 4 * (int64_t)j;
                const float gl[3] = {(float)gd[0], (float)gd[1], (float)gd[2]};
                const float r = sqrt32(pg.sx * pg.sx + pg.sy * pg.sy + pg.sz * pg.sz);
                ivanova_surface32(pg.sx, pg.sy, pg.sz, r, iHk, rk[F_V], gk, rl[F_IH], rl[F_V], gl,
                                  pg.Ax, pg.Ay, pg.Az);
                pg.An = sqrt32(pg.Ax * pg.Ax + pg.Ay * pg.Ay + pg.Az * pg.Az);
            }
            const float dtVl = dtf * rcp32(rl[F_V]);
            const bool use = valid && pg.An > 0.0f;
            // the stages in program order (see the transport)
            __builtin_amdgcn_sched_barrier(0);
            store_rows32(v, sb, lane);          // the record rows
            {                                   // the next iteration's geometry rows
#pragma unroll
                for (int m = 0; m < 4; ++m) row[m] = __shfl(jn, 16 * m + (lane >> 2), 64);
                load_rows32<OFF32>(geo32, row, lane, v);
            }
            const Row32 Rl(sb, lane);
            float qLp[4], qRp[4], qL[4], qR[4];
            bool own_slope[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                const float dk = Di[3 * m] * pg.sx + Di[3 * m + 1] * pg.sy + Di[3 * m + 2] * pg.sz;
                const float dl = Rl[4 + 3 * m] * pg.sx + Rl[5 + 3 * m] * pg.sy + Rl[6 + 3 * m] * pg.sz;
                const float mm = minmod32(dk, dl);
                own_slope[m] = (dk * dl > 0.0f) && (fabsf(dk) <= fabsf(dl));
                qLp[m] = qL[m] = Ui[m] + pg.fk * mm;
                qRp[m] = qR[m] = Rl[m] - pg.fl * mm;
            }
            guard32(qL[0], qL[1], qL[2], qL[3], cf);
            guard32(qR[0], qR[1], qR[2], qR[3], cf);
            const float Llm[4] = {Ll.x, Ll.y, Ll.z, Ll.w};
            float nu[4], tL[4], tR[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) nu[m] = 0.5f * (dtVl * Llm[m] - dtVk * Li[m]);
            m1_flux32_vjp(qL[0], qL[1], qL[2], qL[3], pg.Ax, pg.Ay, pg.Az, c2, ic2, nu, tL);
            m1_flux32_vjp(qR[0], qR[1], qR[2], qR[3], pg.Ax, pg.Ay, pg.Az, c2, ic2, nu, tR);
            if constexpr (HLL) {
                const float iAn = pg.An > 0.0f ? rcp32(pg.An) : 0.0f;
                float loL, hiL, loR, hiR, w1, w2, w3;
                hll_speeds32(qL[0], qL[1], qL[2], qL[3], pg.Ax, pg.Ay, pg.Az, iAn, cf, ic2, hll,
                             loL, hiL);
                hll_speeds32(qR[0], qR[1], qR[2], qR[3], pg.Ax, pg.Ay, pg.Az, iAn, cf, ic2, hll,
                             loR, hiR);
                hll_weights32(loL, hiL, loR, hiR, pg.An, w1, w2, w3);
                float FL[4], FR[4];
                m1_flux32(qL[0], qL[1], qL[2], qL[3], pg.Ax, pg.Ay, pg.Az, c2, ic2, FL);
                m1_flux32(qR[0], qR[1], qR[2], qR[3], pg.Ax, pg.Ay, pg.Az, c2, ic2, FR);
                float S1 = 0.0f, S2 = 0.0f, S3 = 0.0f;   // m . (F_L, F_R, U_R - U_L)
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    S1 += nu[m] * FL[m];
                    S2 += nu[m] * FR[m];
                    S3 += nu[m] * (qR[m] - qL[m]);
                    tL[m] = 2.0f * (w1 * tL[m] - w3 * nu[m]);
                    tR[m] = 2.0f * (w2 * tR[m] + w3 * nu[m]);
                }
                float gloL, ghiL, gloR, ghiR;
                hll_weights32_vjp(loL, hiL, loR, hiR, pg.An, 2.0f * S1, 2.0f * S2, 2.0f * S3,
                                  gloL, ghiL, gloR, ghiR);
                hll_speeds32_vjp(qL[0], qL[1], qL[2], qL[3], pg.Ax, pg.Ay, pg.Az, iAn, cf, ic2,
                                 hll, gloL, ghiL, tL);
                hll_speeds32_vjp(qR[0], qR[1], qR[2], qR[3], pg.Ax, pg.Ay, pg.Az, iAn, cf, ic2,
                                 hll, gloR, ghiR, tR);
            } else {
                const float dis = cf * pg.An;
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    tL[m] += dis * nu[m];
                    tR[m] -= dis * nu[m];
                }
            }
            guard32_vjp(qLp, tL, cf);
            guard32_vjp(qRp, tR, cf);
            float lm[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) lm[m] = own_slope[m] ? pg.fk * tL[m] - pg.fl * tR[m] : 0.0f;
            // the quad's four pairs in list order, component sub
            quad_transpose(tL, sub);
            quad_transpose(lm, sub);
            auto add = [&](int on, float t, float l, float x, float y, float z) {
                if (on) {
                    aU.add(t);
                    aD[0] += l * x;
                    aD[1] += l * y;
                    aD[2] += l * z;
                }
            };
            add(quad_bcast<0>((int)use), tL[0], lm[0], quad_bcast<0>(pg.sx), quad_bcast<0>(pg.sy), quad_bcast<0>(pg.sz));
            add(quad_bcast<1>((int)use), tL[1], lm[1], quad_bcast<1>(pg.sx), quad_bcast<1>(pg.sy), quad_bcast<1>(pg.sz));
            add(quad_bcast<2>((int)use), tL[2], lm[2], quad_bcast<2>(pg.sx), quad_bcast<2>(pg.sy), quad_bcast<2>(pg.sz));
            add(quad_bcast<3>((int)use), tL[3], lm[3], quad_bcast<3>(pg.sx), quad_bcast<3>(pg.sy), quad_bcast<3>(pg.sz));
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if (!active) return;
    const float iV = rcp32(rk[F_V]);
    const float b00 = Bk[0] * iV, b01 = Bk[1] * iV, b02 = Bk[2] * iV;
    const float b11 = Bk[3] * iV, b12 = Bk[4] * iV, b22 = Bk[5] * iV;
    float *o = R + (i * G + g0) * 16;
    o[sub] = (float)((double)(sub == 0 ? +Li[0] : sub == 1 ? +Li[1] : sub == 2 ? +Li[2] : +Li[3]) +
                     aU.value());
    o[4 + 3 * sub + 0] = b00 * aD[0] + b01 * aD[1] + b02 * aD[2];
    o[4 + 3 * sub + 1] = b01 * aD[0] + b11 * aD[1] + b12 * aD[2];
    o[4 + 3 * sub + 2] = b02 * aD[0] + b12 * aD[1] + b22 * aD[2];
}

// Q lanes share a particle, each taking every Q-th neighbour slot; the
// per-lane compensated sums are combined in FP64 by a fixed butterfly.
template <int G, int Q, bool OFF32>
__global__ __launch_bounds__(kBlock) void k_adj_grad32(
    int64_t n, int64_t nb, const float *__restrict__ geo32, const int32_t *__restrict__ nbr,
    const int64_t *__restrict__ wave_base, const int32_t *__restrict__ n_nbr,
    const float *__restrict__ R, float *__restrict__ lam, double box) {
    static_assert(Q == 1 || Q == 2 || Q == 4, "lanes per particle: 1, 2 or 4");
    constexpr int NQ = 4 * G, PW = 64 / Q, PB = kBlock / Q;
    __shared__ __attribute__((aligned(16))) float stage[kBlock / 64][64 * kStage32];
    const int64_t blk = xcd_block(nb);
    if (blk >= nb) return;
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
    const int sub = lane % Q;
    const int64_t i0 = blk * PB + wv * PW;      // first particle of the wave
    const int64_t i = i0 + lane / Q;
    const bool active = i < n;
    const bool owner = active && sub == 0;
    const int64_t ic = active ? i : n - 1;
    const int64_t w = i0 >> 6;
    const bool wave_live = i0 < n;
    const double ibox = 1.0 / box;
    float *sb = stage[wv];
    const float *rp = geo32 + (int64_t)F_REC * ic;
    const double *xp = reinterpret_cast<const double *>(rp);
    const double px = xp[0], py = xp[1], pz = xp[2];
    const float iHp = rp[F_IH];
    Kahan acc[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) acc[q].s = acc[q].c = 0.0f;
    float sgx = 0.0f, sgy = 0.0f, sgz = 0.0f;
    if (wave_live) {
        const int64_t base = wave_base[w] + (i & 63);
        int32_t kmax = (int32_t)((wave_base[w + 1] - wave_base[w]) >> 6);
        const int32_t nn = active ? n_nbr[i] : 0;
        if (Q > 1) {                            // the longest list of this wave's particles
            kmax = nn;
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) kmax = max(kmax, __shfl_xor(kmax, o, 64));
        }
        // the next iteration's neighbour index is loaded one iteration ahead
        int32_t jn = sub < nn ? nbr[base + 64 * (int64_t)sub] : (int32_t)ic;
        for (int32_t kk = 0; kk < kmax; kk += Q) {
            const int32_t k = kk + sub;
            const bool valid = k < nn;
            const int32_t j = jn;
            jn = k + Q < nn ? nbr[base + 64 * (int64_t)(k + Q)] : (int32_t)ic;
            uint32_t row[4];
#pragma unroll
            for (int m = 0; m < 4; ++m) row[m] = __shfl(j, 16 * m + (lane >> 2), 64);
            // all rows of this slot in flight before the first is staged
            constexpr int GC = G < 6 ? G : 6;
            fvec4 vp[4], vr[GC][4];
            load_rows32<OFF32>(geo32, row, lane, vp);
#pragma unroll
            for (int g = 0; g < GC; ++g) {
                uint32_t rowg[4];
#pragma unroll
                for (int m = 0; m < 4; ++m) rowg[m] = row[m] * G + g;
                load_rows32<OFF32>(R, rowg, lane, vr[g]);
            }
            store_rows32(vp, sb, lane);
            const Row32 rl(sb, lane);
            const double xl[3] = {rl.pos(0), rl.pos(1), rl.pos(2)};
            const float sx = (float)min_image(xl[0] - px, box, ibox);
            const float sy = (float)min_image(xl[1] - py, box, ibox);
            const float sz = (float)min_image(xl[2] - pz, box, ibox);
            const float r = sqrt32(sx * sx + sy * sy + sz * sz);
            const float wpi = valid ? kern_wf(r * iHp) : 0.0f;
            const float wip = valid ? kern_wf(r * rl[F_IH]) : 0.0f;
            sgx += wpi * sx;
            sgy += wpi * sy;
            sgz += wpi * sz;
#pragma unroll
            for (int c0 = 0; c0 < G; c0 += GC) {
                if (c0 > 0) {
#pragma unroll
                    for (int g = 0; g < GC; ++g) {
                        if (c0 + g >= G) break;
                        uint32_t rowg[4];
#pragma unroll
                        for (int m = 0; m < 4; ++m) rowg[m] = row[m] * G + c0 + g;
                        load_rows32<OFF32>(R, rowg, lane, vr[g]);
                    }
                }
#pragma unroll
                for (int g = 0; g < GC; ++g) {
                    if (c0 + g >= G) break;
                    store_rows32(vr[g], sb, lane);
                    const Row32 Rl(sb, lane);
#pragma unroll
                    for (int m = 0; m < 4; ++m)
                        acc[4 * (c0 + g) + m].add(
                            -wip * (Rl[4 + 3 * m] * sx + Rl[5 + 3 * m] * sy + Rl[6 + 3 * m] * sz));
                }
            }
        }
    }
    double av[NQ];
#pragma unroll
    for (int q = 0; q < NQ; ++q) av[q] = acc[q].value();
    if (Q > 1) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) quad_sum<Q>(av[q]);
        quad_sum<Q>(sgx);
        quad_sum<Q>(sgy);
        quad_sum<Q>(sgz);
    }
    if (!owner) return;
#pragma unroll
    for (int g = 0; g < G; ++g) {
        const float *Rp = R + (i * G + g) * 16;
#pragma unroll
        for (int m = 0; m < 4; ++m)
            lam[(i * G + g) * 4 + m] = (float)(
                (double)Rp[m] - (double)(sgx * Rp[4 + 3 * m] + sgy * Rp[5 + 3 * m] + sgz * Rp[6 + 3 * m]) +
                av[4 * g + m]);
    }
}

// Lanes per particle of the FP32 transposed gradient (1, 2 or 4); 4 took the
// FP32C backward of the 128^3 adjoint workload from 188 to 166 ms.
#ifndef RT_ADJ32_GRAD_Q
#define RT_ADJ32_GRAD_Q 4
#endif
constexpr int kAGQ32 = RT_ADJ32_GRAD_Q;

template <int G>
void launch(rt_ctx *ctx, const float *UD, const float *Uung, const float *lam_next, float *lam2,
            float *R, float *lam, const double *dt) {
    const int64_t n = ctx->p.n, nt = ctx->nwaves;
    hipStream_t st = ctx->stream;
    k_adj_guard32<G><<<nblk(n * G), kBlock, 0, st>>>(n, Uung, lam_next, lam2, (float)ctx->p.c_red);
    const float2 *tab = (const float2 *)ctx->hll_table32;
    const bool iva = ctx->surfaces == RT_IVANOVA;
    // rows addressed by 32-bit offsets while the gradient records fit 4 GiB
    const bool off32 = (uint64_t)n * 64u * G < (uint64_t(1) << 32);
#define RT_ADJ32_PAIR_LAUNCH_O(OFF32_, HLL_, IVA_)                                             \
    k_adj_pair32<OFF32_, HLL_, IVA_><<<(unsigned)xcd_grid(nt * G), kBlock, 0, st>>>(           \
        n, nt, G, ctx->geo32, ctx->geo, ctx->nbr, ctx->wave_base, ctx->n_nbr, UD, lam2, dt,    \
        ctx->p.c_red, ctx->p.box, R, tab, ctx->ivan)
#define RT_ADJ32_PAIR_LAUNCH(HLL_, IVA_)                                                       \
    do {                                                                                       \
        if (off32) RT_ADJ32_PAIR_LAUNCH_O(true, HLL_, IVA_);                                   \
        else RT_ADJ32_PAIR_LAUNCH_O(false, HLL_, IVA_);                                        \
    } while (0)
    if (ctx->solver == RT_HLL) {
        if (iva) RT_ADJ32_PAIR_LAUNCH(true, true);
        else RT_ADJ32_PAIR_LAUNCH(true, false);
    } else {
        if (iva) RT_ADJ32_PAIR_LAUNCH(false, true);
        else RT_ADJ32_PAIR_LAUNCH(false, false);
    }
#undef RT_ADJ32_PAIR_LAUNCH
#undef RT_ADJ32_PAIR_LAUNCH_O
    const int64_t ng = (n + kBlock / kAGQ32 - 1) / (kBlock / kAGQ32);
    if (off32)
        k_adj_grad32<G, kAGQ32, true><<<(unsigned)xcd_grid(ng), kBlock, 0, st>>>(
            n, ng, ctx->geo32, ctx->nbr, ctx->wave_base, ctx->n_nbr, R, lam, ctx->p.box);
    else
        k_adj_grad32<G, kAGQ32, false><<<(unsigned)xcd_grid(ng), kBlock, 0, st>>>(
            n, ng, ctx->geo32, ctx->nbr, ctx->wave_base, ctx->n_nbr, R, lam, ctx->p.box);
}

}  // namespace

void rt_adjoint32(rt_ctx *ctx, const float *UD, const float *Uung, const float *lam_next,
                  float *lam2, float *R, float *lam, const double *dt) {
    switch (ctx->p.groups) {
        case 1: launch<1>(ctx, UD, Uung, lam_next, lam2, R, lam, dt); break;
        case 2: launch<2>(ctx, UD, Uung, lam_next, lam2, R, lam, dt); break;
        case 3: launch<3>(ctx, UD, Uung, lam_next, lam2, R, lam, dt); break;
        case 4: launch<4>(ctx, UD, Uung, lam_next, lam2, R, lam, dt); break;
        case 5: launch<5>(ctx, UD, Uung, lam_next, lam2, R, lam, dt); break;
        case 6: launch<6>(ctx, UD, Uung, lam_next, lam2, R, lam, dt); break;
        case 7: launch<7>(ctx, UD, Uung, lam_next, lam2, R, lam, dt); break;
        case 8: launch<8>(ctx, UD, Uung, lam_next, lam2, R, lam, dt); break;
        default: break;
    }
}
