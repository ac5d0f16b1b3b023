// Head of a V-cycle on a small periodic level in one launch (Sec. III.C): residual
// of the smoothed state, 8-child averages to the coarse level, and the coarse
// right-hand side f^H = L^H(R u) - R d.  A block owns a BB^3 brick, i.e. a
// (BB/2)^3 coarse brick, and stages the state on a two-cell ring: its cells'
// residuals need one ring cell, and the averages on a one-cell coarse ring, which
// the coarse operator needs, take two fine ones (recomputed, not exchanged).
//
// On levels of at most BRICK_CELLS cells the separate residual and coarse
// right-hand-side passes cost 6-7 us each, nearly all launch, first-load and
// reduction latency, besides 1-2 us between dependent launches; together they take
// 4.6-6.8 us (FP64 and FP32 correction, 16^3 to 64^3).  The level's cbar is not
// worth a launch either (the reduction took 4-5 us): its sums go to the next brick
// sweep or coarse tail (PendingCbar).  At 128^3 the rings' extra loads outweigh
// this (whole solves: 128^3 mixed 2.00 ms with the head on its finest level, 1.88
// without; 256^3 FP64 10.25 and 10.10 ms), hence HEAD_CELLS.
//
// Policy interface:
//   K::T, K::Cell           value type; what a cell holds (T phi, or float2 (e, phi~))
//   k.load_cell(i), k.load_src(i)   element i of the fine level
//   k.load_csrc(ci)         per-cell sources of the coarse level
//   k.residual(v, centre, src, acc)  d of a cell from its 18 neighbours; adds the
//                           pass's sums to acc
//   k.coarse(v, centre, rd, rf, csrc, ci, acc)   forms and stores a coarse cell (rd,
//                           rf: averages of d and, with norms, of the fine source)
//   k.pair(a, b), k.eighth(s)   sums and averages of cells
#pragma once

#include "brick.h"

namespace vmg {

constexpr int HEAD_NT = BB * BB * BB;

// part / part_c receive the block's sums of the fine and of the coarse pass: with
// NORM a row of R_NSLOT, else the one value that cbar takes, the sum of Q and f
template <bool NORM, typename K>
__device__ __forceinline__ void head_brick(const K& k, const Geom& g, const Geom& gc, int bx0, int by0, int bz0,
                                           double* part, double* part_c) {
    using T = typename K::T;
    using Cell = typename K::Cell;
    constexpr int RW = BB + 4, RW2 = RW * RW, NU = RW2 * RW, NL = (NU + HEAD_NT - 1) / HEAD_NT;
    constexpr int CB = BB / 2, CW = CB + 2, CW2 = CW * CW, NC = CW2 * CW;
    static_assert(CB * CB * CB == 64 && NC <= HEAD_NT / 2, "one wave of coarse cells; their ring on half the block");
    __shared__ Cell U[NU], C[NC];
    __shared__ T D[HEAD_NT], F[NORM ? HEAD_NT : 1];
    __shared__ double red[HEAD_NT / 64][NORM ? R_NSLOT : 1];
    const int tid = threadIdx.x;
    const int x = tid % BB, y = (tid / BB) % BB, z = tid / (BB * BB);      // this thread's cell of the brick
    const bool ok = bx0 + x < g.n0 && by0 + y < g.n1 && bz0 + z < g.n2;
    const int I = tid % CB, J = (tid / CB) % CB, Z = tid / (CB * CB);      // first wave: its coarse cell
    const int cx = bx0 / 2 + I, cy = by0 / 2 + J, cz = bz0 / 2 + Z;
    const bool cok = tid < 64 && cx < gc.n0 && cy < gc.n1 && cz < gc.n2;
    // every load is issued before the first LDS write
    Cell u0[NL];
#pragma unroll
    for (int q = 0; q < NL; ++q) {
        const int e = tid + q * HEAD_NT;
        if (e < NU)
            u0[q] = k.load_cell(small_index<0>(g, wrapi(bx0 - 2 + e % RW, g.n0), wrapi(by0 - 2 + (e / RW) % RW, g.n1),
                                               wrapi(bz0 - 2 + e / RW2, g.n2)));
    }
    typename K::Src src{};
    if (ok) src = k.load_src(small_index<0>(g, bx0 + x, by0 + y, bz0 + z));
    typename K::CSrc csrc{};
    const int64_t ci = cok ? small_index<0>(gc, cx, cy, cz) : 0;
    if (cok) csrc = k.load_csrc(ci);
#pragma unroll
    for (int q = 0; q < NL; ++q) {
        const int e = tid + q * HEAD_NT;
        if (e < NU) U[e] = u0[q];
    }
    __syncthreads();
    double acc[R_NSLOT] = {0, 0, 0, 0, 0, 0, 0};
    if (ok) {
        const int c = ((z + 2) * RW + y + 2) * RW + x + 2;
        NbT<Cell> v;
        brick_nb<RW>(U, c, v);
        D[tid] = k.residual(v, U[c], src, acc);
        if constexpr (NORM) F[tid] = src.f;
    }
    // averages on the coarse brick's ring (children paired along x, y, then z)
    const int ct = tid - HEAD_NT / 2;
    if (ct >= 0 && ct < NC) {
        const int b = ((2 * (ct / CW2)) * RW + 2 * ((ct / CW) % CW)) * RW + 2 * (ct % CW);
        auto quad = [&](int o) { return k.pair(k.pair(U[o], U[o + 1]), k.pair(U[o + RW], U[o + RW + 1])); };
        C[ct] = k.eighth(k.pair(quad(b), quad(b + RW2)));
    }
    __syncthreads();
    if (tid < 64) {
        double acc_c[R_NSLOT] = {0, 0, 0, 0, 0, 0, 0};
        if (cok) {
            const int b = ((2 * Z) * BB + 2 * J) * BB + 2 * I;
            auto avg = [&](const T* a) {
                auto quad = [&](int o) { return (a[o] + a[o + 1]) + (a[o + BB] + a[o + BB + 1]); };
                return T(0.125) * (quad(b) + quad(b + BB * BB));
            };
            const T rd = avg(D), rf = NORM ? avg(F) : T(0);
            const int c = ((Z + 1) * CW + J + 1) * CW + I + 1;
            NbT<Cell> v;
            brick_nb<CW>(C, c, v);
            k.coarse(v, C[c], rd, rf, csrc, ci, acc_c);
        }
        if (NORM) {
            double* out = part_c + (int64_t)blockIdx.x * R_NSLOT;
            const double q = wave_sum(acc_c[R_Q]), f = wave_sum(acc_c[R_F]);
            const double d1 = wave_sum(acc_c[R_D1]), d2 = wave_sum(acc_c[R_D2]);
            if (tid == 0) {
                out[R_Q] = q;
                out[R_F] = f;
                out[R_D1] = d1;
                out[R_D2] = d2;
            }
        } else {
            const double qf = wave_sum(acc_c[R_Q] + acc_c[R_F]);
            if (tid == 0) part_c[blockIdx.x] = qf;
        }
    }
    const int lane = tid & 63, w = tid >> 6;
    if (NORM) {
#pragma unroll
        for (int s = 0; s < R_NSLOT; ++s) {
            const double t = wave_sum(acc[s]);
            if (lane == 0) red[w][s] = t;
        }
    } else {
        const double qf = wave_sum(acc[R_Q] + acc[R_F]);
        if (lane == 0) red[w][0] = qf;
    }
    __syncthreads();
    if (tid < (NORM ? R_NSLOT : 1)) {
        double s = 0.0;
#pragma unroll
        for (int q = 0; q < HEAD_NT / 64; ++q) s += red[q][tid];
        part[(int64_t)blockIdx.x * (NORM ? R_NSLOT : 1) + tid] = s;
    }
}

}  // namespace vmg
