// Coarse tail of a periodic V-cycle (Sec. III.C): every level with at most
// TAIL_CELLS cells, down to the coarsest, in one single-workgroup launch with the
// state in LDS.  On these grids a separate launch per step costs more than the
// step itself.  A periodic level coarsens only while every axis keeps 4 cells,
// so the tail is either 8^3 and 4^3 (k_tail8) or one coarsest level of any shape
// (k_tail1).
//
// The arithmetic is the multi-kernel V-cycle's, step for step:
//   * fused red-black sweep with snapshot semantics (red from the old state,
//     black from the red-updated one), in place: each colour is computed into
//     registers, then written after a barrier;
//   * residual d = L(phi) - f + cbar, 8-child averages of phi and d, then
//     cbar <- (sum f + sum Q) / N for the level's later sweeps;
//   * coarse rhs f^H = L^H(R phi) - R d;
//   * coarsest level: cbar from the current sum of Q before every sweep;
//   * cell-centred trilinear prolongation of phi^H - R phi (periodic wrap).
// Reductions run in a fixed order, so results are bitwise reproducible.
//
// What bounds it: a serial chain of some 20 colour phases on one CU.  Each
// thread therefore owns its cells for the whole launch (values, right-hand side
// and per-cell constants in registers, neighbour offsets from compile-time
// sizes), so a phase is 18 LDS reads, one root and one LDS write; the 8^3 level
// runs on four waves (one cell of each colour per thread), and 4^3 on one wave,
// whose phases need no barrier; sums across a wave use DPP adds.
// 8^3 over 4^3 with V(2,2) and 4 (8) coarsest sweeps: FP64 8.4 (10.9) us, FP32
// correction 9.2 us; with 512 threads, run-time sizes, a barrier per step on both
// levels and values re-read from LDS it took 23.3 (32.8) and 26.8 us.
#include <hip/hip_runtime.h>

#include "brick.h"

namespace vmg {

namespace {

// LDS written by a lane of this wave is read by another after this: the LDS
// serves a wave's accesses in order, so only the compiler has to keep them so.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Offsets of a cell and its two neighbours along each axis ([0] = -1, [1] = the
// cell, [2] = +1) with periodic wrap: a neighbour's index is the sum of three.
struct TNbr {
    int x[3], y[3], z[3];
    __device__ __forceinline__ int centre() const { return z[1] + y[1] + x[1]; }
};

__device__ __forceinline__ TNbr tail_nbr(int n0, int n1, int n2, int i, int j, int k) {
    TNbr o;
    const int p = n0 * n1;
    o.x[0] = i == 0 ? n0 - 1 : i - 1;
    o.x[1] = i;
    o.x[2] = i == n0 - 1 ? 0 : i + 1;
    o.y[0] = (j == 0 ? n1 - 1 : j - 1) * n0;
    o.y[1] = j * n0;
    o.y[2] = (j == n1 - 1 ? 0 : j + 1) * n0;
    o.z[0] = (k == 0 ? n2 - 1 : k - 1) * p;
    o.z[1] = k * p;
    o.z[2] = (k == n2 - 1 ? 0 : k + 1) * p;
    return o;
}

template <typename T>
__device__ __forceinline__ void tail_gather(const TNbr& o, const T* u, NbT<T>& v) {
    auto at = [&](int a, int b, int c) { return u[o.z[c] + o.y[b] + o.x[a]]; };
    v.xm = at(0, 1, 1);   v.xp = at(2, 1, 1);
    v.ym = at(1, 0, 1);   v.yp = at(1, 2, 1);
    v.zm = at(1, 1, 0);   v.zp = at(1, 1, 2);
    v.xpyp = at(2, 2, 1); v.xmym = at(0, 0, 1); v.xpym = at(2, 0, 1); v.xmyp = at(0, 2, 1);
    v.xpzp = at(2, 1, 2); v.xmzm = at(0, 1, 0); v.xpzm = at(2, 1, 0); v.xmzp = at(0, 1, 2);
    v.ypzp = at(1, 2, 2); v.ymzm = at(1, 0, 0); v.ypzm = at(1, 2, 0); v.ymzp = at(1, 0, 2);
}

// The FP64 problem: per-cell constant delta.
struct TailK {
    using T = double;
    static constexpr bool BASE = false;   // no base state phi~
    struct Cell {
        double del;
    };
    Coef c;
    double h2, inv_h2, inv_h4;   // of one level
    float kk;
    __device__ TailK(const Coef& c_, double h) : c(c_) {
        h2 = h * h;
        inv_h2 = 1.0 / h2;
        inv_h4 = inv_h2 * inv_h2;
        kk = kink_k(h2);
    }
    __device__ void batch_coefs(double) {}
    // root Q of a cell, its neighbour sum S and discriminant D
    __device__ double root(const NbT<double>& v, const Cell& k, double& S, double& D) const {
        return nl_root_d(v, k.del, c, inv_h4, S, D);
    }
};

// The mixed path's FP32 correction problem Lap e - dQ(e) = r - cbar_e: the base
// state phi~ enters through six differences of its neighbours, which stay fixed
// over the launch, and t0 = +-sqrt|D0|.
struct TailCorrK {
    using T = float;
    static constexpr bool BASE = true;
    struct Cell {
        float dxy, dxz, dyz, bxy, bxz, byz;   // 2 x the differences of phi~
        float t0;
    };
    CoefF c;
    Coef c64;
    float h2, inv_h2, a_ih4;
    double inv_h4;
    float kk;
    __device__ TailCorrK(const Coef& c_, double h) : c64(c_) {
        c.alpha = (float)c_.alpha;
        c.c8 = (float)c_.c8;
        c.a34 = c_.alpha != 0.0 ? (float)(3.0 / (4.0 * c_.alpha)) : 0.0f;
        const double hh = h * h;
        h2 = (float)hh;
        inv_h2 = (float)(1.0 / hh);
        inv_h4 = 1.0 / (hh * hh);
        a_ih4 = (float)(c_.alpha * inv_h4);
        kk = kink_k(h2);
    }
    // the coefficients as the batched passes round them
    __device__ void batch_coefs(double h) { a_ih4 = c.alpha / (float)(h * h * h * h); }
    __device__ static void base_cell(const NbT<float>& p, Cell& k) {
        const float sx = p.xp + p.xm, sy = p.yp + p.ym, sz = p.zp + p.zm;
        k.dxy = 2.0f * (sx - sy);
        k.dxz = 2.0f * (sx - sz);
        k.dyz = 2.0f * (sy - sz);
        k.bxy = 2.0f * ((p.xpyp + p.xmym) - (p.xpym + p.xmyp));
        k.bxz = 2.0f * ((p.xpzp + p.xmzm) - (p.xpzm + p.xmzp));
        k.byz = 2.0f * ((p.ypzp + p.ymzm) - (p.ypzm + p.ymzp));
    }
    // +-sqrt|D0| from the FP64 discriminant of phi~ and the density
    __device__ float base_t0(const NbT<float>& p, double del) const {
        Nb v;
        v.xm = p.xm; v.xp = p.xp; v.ym = p.ym; v.yp = p.yp; v.zm = p.zm; v.zp = p.zp;
        v.xpyp = p.xpyp; v.xmym = p.xmym; v.xpym = p.xpym; v.xmyp = p.xmyp;
        v.xpzp = p.xpzp; v.xmzm = p.xmzm; v.xpzm = p.xpzm; v.xmzp = p.xmzp;
        v.ypzp = p.ypzp; v.ymzm = p.ymzm; v.ypzm = p.ypzm; v.ymzp = p.ymzp;
        const double D0 = base_discriminant(v, del, c64, inv_h4);
        return (float)(D0 >= 0.0 ? sqrt(D0) : -sqrt(-D0));
    }
    __device__ float root(const NbT<float>& e, const Cell& k, float& Se, float& D1) const {
        const float sx = e.xp + e.xm, sy = e.yp + e.ym, sz = e.zp + e.zm;
        Se = sx + sy + sz;
        const float dxy = sx - sy, dxz = sx - sz, dyz = sy - sz;
        const float bxy = (e.xpyp + e.xmym) - (e.xpym + e.xmyp);
        const float bxz = (e.xpzp + e.xmzm) - (e.xpzm + e.xmzp);
        const float byz = (e.ypzp + e.ymzm) - (e.ypzm + e.ymzp);
        const float pd = fmaf(k.dxy + dxy, dxy, fmaf(k.dxz + dxz, dxz, (k.dyz + dyz) * dyz));
        const float pb = fmaf(k.bxy + bxy, bxy, fmaf(k.bxz + bxz, bxz, (k.byz + byz) * byz));
        return dQ_of_d(fmaf(a_ih4 * (1.0f / 3.0f), pd, a_ih4 * 0.125f * pb), k.t0, c, D1);
    }
};

// updated value of a cell (old value `old`, right-hand side f)
template <typename K, typename T>
__device__ __forceinline__ T tail_update(const K& k, const NbT<T>& v, const typename K::Cell& cell, T old, T f, T cb) {
    T S, D;
    const T Q = k.root(v, cell, S, D);
    return kink_relax(old, (S - k.h2 * (Q + f - cb)) * T(1.0 / 6.0), D, k.kk);
}

constexpr int T8_NT = 256;

}  // namespace

// Arguments common to both problems (launch_tail, launch_tail_corr fill them).
template <typename T>
struct Tail {
    int n[3];               // top level's cells
    double h;               // its cell size
    const double* delta;    // its density (FP64 problem)
    const double* delta_c;  // density of the 4^3 level (k_tail8)
    T* u;                   // its state (in/out)
    const T* f;             // its right-hand side (may be null: zero)
    const T *pt, *t0;       // correction problem: base state and +-sqrt|D0|
    LevelScalars* sc;       // its cbar (in/out)
    PendingCbar pend;       // ... or the sums it is still in
    Coef c;
    int nu1, nu2, ncoarse;
};

// 8^3 over 4^3.
template <typename K>
__global__ void __launch_bounds__(T8_NT) k_tail8(Tail<typename K::T> a) {
    using T = typename K::T;
    __shared__ T u8[512], d8[512], pt8[K::BASE ? 512 : 1];
    __shared__ T u4[64], c4[64], pt4[K::BASE ? 64 : 1];
    __shared__ double red[T8_NT / 64][2], psum;
    const int tid = threadIdx.x;
    const K k8(a.c, a.h), k4(a.c, 2.0 * a.h);
    // this thread's cells of the 8^3 level: colour 0 and 1 of one x pair of a row
    const int j8 = (tid >> 2) & 7, z8 = tid >> 5;
    TNbr o8[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) o8[q] = tail_nbr(8, 8, 8, 2 * (tid & 3) + ((j8 + z8 + q) & 1), j8, z8);
    T v8[2], f8[2];
    typename K::Cell g8[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int e = o8[q].centre();
        v8[q] = a.u[e];
        f8[q] = a.f ? a.f[e] : T(0);
        if constexpr (K::BASE) {
            g8[q].t0 = a.t0[e];
            pt8[e] = a.pt[e];
        } else {
            g8[q].del = a.delta[e];
        }
    }
    // the 4^3 level: one cell per lane of the first wave
    const TNbr o4 = tail_nbr(4, 4, 4, tid & 3, (tid >> 2) & 3, (tid >> 4) & 3);
    const double del4 = tid < 64 ? a.delta_c[tid] : 0.0;
    double share = 0.0;
    T cb8 = T(0);
    if (!a.pend.part) cb8 = (T)a.sc->cbar;
    else if (tid < 64) share = pending_share(a.pend);
#pragma unroll
    for (int q = 0; q < 2; ++q) u8[o8[q].centre()] = v8[q];
    if (a.pend.part && tid < 64) {
        share = wave_sum(share);
        if (tid == 0) psum = share;
    }
    __syncthreads();
    if (a.pend.part) cb8 = (T)(psum / 512.0);
    if constexpr (K::BASE) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            NbT<T> p;
            tail_gather(o8[q], pt8, p);
            K::base_cell(p, g8[q]);
        }
    }
    auto sweeps8 = [&](int count) {
        for (int s = 0; s < count; ++s)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                NbT<T> v;
                tail_gather(o8[q], u8, v);
                v8[q] = tail_update(k8, v, g8[q], v8[q], f8[q], cb8);
                __syncthreads();
                u8[o8[q].centre()] = v8[q];
                __syncthreads();
            }
    };
    sweeps8(a.nu1);
    // residual of every 8^3 cell, then the level's new cbar
    double sq = 0.0, sf = 0.0;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        NbT<T> v;
        tail_gather(o8[q], u8, v);
        T S, D;
        const T Q = k8.root(v, g8[q], S, D);
        d8[o8[q].centre()] = (S - T(6) * v8[q]) * k8.inv_h2 - Q - f8[q] + cb8;
        sq += Q;
        sf += f8[q];
    }
    sq = wave_sum(sq);
    sf = wave_sum(sf);
    if ((tid & 63) == 0) {
        red[tid >> 6][0] = sq;
        red[tid >> 6][1] = sf;
    }
    __syncthreads();
    double SQ = 0.0, SF = 0.0;
#pragma unroll
    for (int w = 0; w < T8_NT / 64; ++w) {
        SQ += red[w][0];
        SF += red[w][1];
    }
    cb8 = (T)((SF + SQ) / 512.0);
    if (tid < 64) {
        // 8-child averages of phi, d (and phi~), children summed in a fixed order
        T su = T(0), sd = T(0), sp = T(0);
        const int I = tid & 3, J = (tid >> 2) & 3, Z = tid >> 4;
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            const int e = ((2 * Z + (m >> 2)) * 8 + 2 * J + ((m >> 1) & 1)) * 8 + 2 * I + (m & 1);
            sd += d8[e];
            su += u8[e];
            if constexpr (K::BASE) sp += pt8[e];
        }
        const T old = T(0.125) * su;
        T v4 = old;
        u4[tid] = v4;
        typename K::Cell g4;
        if constexpr (K::BASE) pt4[tid] = T(0.125) * sp;
        wave_sync();
        if constexpr (K::BASE) {
            NbT<T> p;
            tail_gather(o4, pt4, p);
            K::base_cell(p, g4);
            g4.t0 = k4.base_t0(p, del4);
        } else {
            g4.del = del4;
        }
        // coarse rhs f^H = L^H(R phi) - R d
        NbT<T> v;
        T S, D;
        tail_gather(o4, u4, v);
        T Q = k4.root(v, g4, S, D);
        const T f4 = (S - T(6) * v4) * k4.inv_h2 - Q - T(0.125) * sd;
        const double sf4 = wave_sum((double)f4);
        // coarsest sweeps, cbar from the current sum of Q before each
        const int colour = (I + J + Z) & 1;
        for (int s = 0; s < a.ncoarse; ++s) {
            tail_gather(o4, u4, v);
            Q = k4.root(v, g4, S, D);
            const T cb = (T)((sf4 + wave_sum((double)Q)) / 64.0);
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                if (colour == q) {
                    tail_gather(o4, u4, v);
                    v4 = tail_update(k4, v, g4, v4, f4, cb);
                }
                wave_sync();
                if (colour == q) u4[tid] = v4;
                wave_sync();
            }
        }
        c4[tid] = v4 - old;
    }
    __syncthreads();
    // prolongation of the correction, post-smoothing
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const int i = o8[q].x[1];
        T acc = T(0);
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            const int ai = m & 1, aj = (m >> 1) & 1, ak = m >> 2;
            const T w = T((ai ? 0.25 : 0.75) * (aj ? 0.25 : 0.75) * (ak ? 0.25 : 0.75));
            const int ci = ((i >> 1) + (ai ? ((i & 1) ? 1 : -1) : 0)) & 3;
            const int cj = ((j8 >> 1) + (aj ? ((j8 & 1) ? 1 : -1) : 0)) & 3;
            const int ck = ((z8 >> 1) + (ak ? ((z8 & 1) ? 1 : -1) : 0)) & 3;
            acc += w * c4[(ck * 4 + cj) * 4 + ci];
        }
        v8[q] += acc;
        u8[o8[q].centre()] = v8[q];
    }
    __syncthreads();
    sweeps8(a.nu2);
#pragma unroll
    for (int q = 0; q < 2; ++q) a.u[o8[q].centre()] = v8[q];
    if (tid == 0) a.sc->cbar = cb8;
}

// One coarsest level of up to 512 cells, any shape: thread t owns cells t and t + NTH.
template <typename K, int NTH>
__global__ void __launch_bounds__(NTH) k_tail1(Tail<typename K::T> a) {
    using T = typename K::T;
    __shared__ T u[TAIL_CELLS], pt[K::BASE ? TAIL_CELLS : 1];
    __shared__ double red[2][NTH / 64];
    const int tid = threadIdx.x;
    const int n0 = a.n[0], n1 = a.n[1], n2 = a.n[2], N = n0 * n1 * n2;
    const K k(a.c, a.h);
    constexpr int NS = NTH >= 256 ? 2 : 1;
    TNbr o[NS];
    T val[NS], f[NS];
    typename K::Cell g[NS];
    int colour[NS];   // -1: no cell
    double sf = 0.0;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int e = tid + s * NTH;
        const bool ok = e < N;
        const int i = ok ? e % n0 : 0, r = ok ? e / n0 : 0, j = r % n1, z = r / n1;
        o[s] = tail_nbr(n0, n1, n2, i, j, z);
        colour[s] = ok ? (i + j + z) & 1 : -1;
        const int c = o[s].centre();
        val[s] = a.u[c];
        f[s] = a.f ? a.f[c] : T(0);
        if constexpr (K::BASE) {
            g[s].t0 = a.t0[c];
            if (ok) pt[e] = a.pt[c];
        } else {
            g[s].del = a.delta[c];
        }
        if (ok) {
            u[e] = val[s];
            sf += f[s];
        }
    }
    __syncthreads();
    if constexpr (K::BASE) {
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            NbT<T> p;
            tail_gather(o[s], pt, p);
            K::base_cell(p, g[s]);
        }
    }
    int turn = 0;   // the two halves of red alternate, so one barrier per sum is enough
    auto total = [&](double x) {
        x = wave_sum(x);
        if (NTH == 64) return x;
        if ((tid & 63) == 0) red[turn][tid >> 6] = x;
        __syncthreads();
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < NTH / 64; ++w) s += red[turn][w];
        turn ^= 1;
        return s;
    };
    const double SF = total(sf);
    for (int sw = 0; sw < a.ncoarse; ++sw) {
        double sq = 0.0;
#pragma unroll
        for (int s = 0; s < NS; ++s)
            if (colour[s] >= 0) {
                NbT<T> v;
                tail_gather(o[s], u, v);
                T S, D;
                sq += k.root(v, g[s], S, D);
            }
        const T cb = (T)((SF + total(sq)) / (double)N);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
#pragma unroll
            for (int s = 0; s < NS; ++s)
                if (colour[s] == q) {
                    NbT<T> v;
                    tail_gather(o[s], u, v);
                    val[s] = tail_update(k, v, g[s], val[s], f[s], cb);
                }
            __syncthreads();
#pragma unroll
            for (int s = 0; s < NS; ++s)
                if (colour[s] == q) u[o[s].centre()] = val[s];
            __syncthreads();
        }
    }
#pragma unroll
    for (int s = 0; s < NS; ++s)
        if (colour[s] >= 0) a.u[o[s].centre()] = val[s];
}

// ---------------------------------------------------------------------------
// Coarse tails of a Dirichlet batch: every grid from its first level of at most 8
// cells per axis down to its coarsest (three levels at most: 8, 4, 2), one
// workgroup per grid, all grids of the batch in one launch at the bottom of the
// cycle, whatever level their tails start on.  Level by level these took 7 to 10
// launches of 5-11 us per level and cycle for a few hundred cells; here a thread
// owns one pair of cells per level, as above, and everything the three levels read
// from memory is requested before the first sweep.  96 grids of 16^3-64^3 (V(1,1),
// FP32 correction): 19 us a cycle, against some 25 launches of 160 us in all.
// The arithmetic is the level-by-level cycle's: ghosts follow the interior
// (reference + odd reflection of the correction) after every sweep, on the
// coarsest level after every colour; the correction prolonged is reflected the
// same way at the faces.
// ---------------------------------------------------------------------------
namespace {

// One level of a tail: cells in an LDS cube of pitch P (ghost shell included),
// run by 256 threads or (WAVE) by one wave.  NG: ghosts per thread.
template <typename K, int P, int NG, bool WAVE>
struct BatchLev {
    using T = typename K::T;
    static constexpr int NTH = WAVE ? 64 : T8_NT;
    K k;
    T* u;
    int n0, n1, n2;
    int i[2], j, z;              // this thread's cells (colour 0 and 1 of a pair)
    int c[2];                    // their LDS elements (-1: none)
    T v[2], f[2];
    typename K::Cell cell[2];
    int gi[NG], gm[NG];          // ghosts: LDS element (-1: none), mirrored interior element
    T gs[NG], og[NG], om[NG];    // sign, reference values of both

    __device__ static int at(int x, int y, int z) { return ((z + 1) * P + y + 1) * P + x + 1; }
    __device__ static void sync() {
        if (WAVE) wave_sync();
        else __syncthreads();
    }
    // (a level the grid does not have comes as 1 x 1 x 0 cells, h = 1)
    __device__ BatchLev(const Coef& coef, const Geom& g, T* lds) : k(coef, g.h), u(lds), n0(g.n0), n1(g.n1), n2(g.n2) {
        k.batch_coefs(g.h);
        const unsigned t = threadIdx.x, h = (unsigned)(n0 + 1) >> 1, r = t / h;
        j = (int)(r % (unsigned)n1);
        z = (int)(r / (unsigned)n1);
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            i[q] = 2 * (int)(t - r * h) + ((j + z + q) & 1);
            c[q] = z < n2 && i[q] < n0 ? at(i[q], j, z) : -1;
            v[q] = f[q] = T(0);
            cell[q] = typename K::Cell{};
        }
    }
    __device__ int64_t element(const Geom& g, int q) const { return small_index<1>(g, i[q], j, z); }
    // ghosts: places, signs and their references from the pool
    __device__ void init_ghosts(const Geom& g, const T* __restrict__ old) {
        const int count = (int)ghost_count_dev(n0, n1, n2);
#pragma unroll
        for (int q = 0; q < NG; ++q) {
            const int e = threadIdx.x + q * NTH;
            gi[q] = -1;
            if (e >= count) continue;
            int x, y, w;
            ghost_coords_t<unsigned>(n0, n1, n2, e, x, y, w);
            int sign = 1;
            const int mx = mirror(x, n0, sign), my = mirror(y, n1, sign), mz = mirror(w, n2, sign);
            gi[q] = at(x, y, w);
            gm[q] = at(mx, my, mz);
            gs[q] = (T)sign;
            og[q] = old[small_index<1>(g, x, y, w)];
        }
    }
    // the references of the mirrored cells: ref(x, y, z), or a cube of this pitch
    template <typename R>
    __device__ void ghost_refs(R&& ref) {
#pragma unroll
        for (int q = 0; q < NG; ++q)
            if (gi[q] >= 0) om[q] = ref(gm[q] % P - 1, (gm[q] / P) % P - 1, gm[q] / (P * P) - 1);
    }
    __device__ void ghost_refs_at(const T* cube) {
#pragma unroll
        for (int q = 0; q < NG; ++q)
            if (gi[q] >= 0) om[q] = cube[gm[q]];
    }
    // ghosts at their references, interior from v
    __device__ void store_all() {
#pragma unroll
        for (int q = 0; q < NG; ++q)
            if (gi[q] >= 0) u[gi[q]] = og[q];
#pragma unroll
        for (int q = 0; q < 2; ++q)
            if (c[q] >= 0) u[c[q]] = v[q];
        sync();
    }
    __device__ void refresh() {
#pragma unroll
        for (int q = 0; q < NG; ++q)
            if (gi[q] >= 0) u[gi[q]] = og[q] + gs[q] * (u[gm[q]] - om[q]);
        sync();
    }
    __device__ void sweeps(int count, bool every_colour) {
        for (int s = 0; s < count; ++s)
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                if (c[q] >= 0) {
                    NbT<T> nb;
                    brick_nb<P>(u, c[q], nb);
                    v[q] = tail_update(k, nb, cell[q], v[q], f[q], T(0));
                }
                sync();
                if (c[q] >= 0) u[c[q]] = v[q];
                sync();
                if (q == 1 || every_colour) refresh();
            }
    }
    // L(u) - f of this thread's cell q
    __device__ T residual(int q) const {
        NbT<T> nb;
        brick_nb<P>(u, c[q], nb);
        T S, D;
        const T Q = k.root(nb, cell[q], S, D);
        return (S - T(6) * v[q]) * k.inv_h2 - Q - f[q];
    }
};

// 8-child average from a fine cube of pitch P, at coarse cell (I, J, Z)
template <int P, typename T>
__device__ __forceinline__ T child_average(const T* a, int I, int J, int Z) {
    T s = T(0);
#pragma unroll
    for (int m = 0; m < 8; ++m)
        s += a[((2 * Z + (m >> 2) + 1) * P + 2 * J + ((m >> 1) & 1) + 1) * P + 2 * I + (m & 1) + 1];
    return T(0.125) * s;
}

// trilinear value at fine cell (x, y, z) of the coarse correction d (cube of pitch
// P), reflected with a sign flip at the faces
template <int P, typename T>
__device__ __forceinline__ T prolong_at(const T* d, int n0, int n1, int n2, int x, int y, int z) {
    T acc = T(0);
#pragma unroll
    for (int m = 0; m < 8; ++m) {
        int sign = 1;
        const int I = mirror((x >> 1) + ((m & 1) ? ((x & 1) ? 1 : -1) : 0), n0, sign);
        const int J = mirror((y >> 1) + ((m & 2) ? ((y & 1) ? 1 : -1) : 0), n1, sign);
        const int Z = mirror((z >> 1) + ((m & 4) ? ((z & 1) ? 1 : -1) : 0), n2, sign);
        const T w = T(((m & 1) ? 0.25 : 0.75) * ((m & 2) ? 0.25 : 0.75) * ((m & 4) ? 0.25 : 0.75));
        acc += w * ((T)sign * d[((Z + 1) * P + J + 1) * P + I + 1]);
    }
    return acc;
}

// phi~ of a level (ghosts included) into an LDS cube of pitch P; all loads first
template <int P, int NTH>
__device__ __forceinline__ void stage_base(const Geom& g, float* cube, const float* __restrict__ pt) {
    constexpr int NL = (P * P * P + NTH - 1) / NTH;
    const int m0 = g.n0 + 2, m1 = g.n1 + 2, n = (int)g.nstore;
    float v[NL];
#pragma unroll
    for (int q = 0; q < NL; ++q) {
        const int e = threadIdx.x + q * NTH;
        v[q] = e < n ? pt[g.base + e] : 0.0f;
    }
#pragma unroll
    for (int q = 0; q < NL; ++q) {
        const int e = threadIdx.x + q * NTH, r = e / m0;
        if (e < n) cube[((r / m1) * P + r % m1) * P + e % m0] = v[q];
    }
}

template <int P, typename L>
__device__ __forceinline__ void base_cells(L& lev, const float* cube) {
#pragma unroll
    for (int q = 0; q < 2; ++q)
        if (lev.c[q] >= 0) {
            NbT<float> p;
            brick_nb<P>(cube, lev.c[q], p);
            TailCorrK::base_cell(p, lev.cell[q]);
        }
}

}  // namespace

template <typename K>
__global__ void __launch_bounds__(T8_NT) k_tail_batch(const TailGrid<typename K::T>* __restrict__ grids, Coef coef,
                                                      int nu1, int nu2, int ncoarse) {
    using T = typename K::T;
    constexpr int PA = 10, PB = 6, PC = 4;
    constexpr int CA = PA * PA * PA, CB = PB * PB * PB, CC = PC * PC * PC;
    __shared__ T uA[CA], dA[CA], oA[CA], uB[CB], dB[CB], uC[CC];
    __shared__ float pA[K::BASE ? CA : 1], pB[K::BASE ? CB : 1], pC[K::BASE ? CC : 1];
    const TailGrid<T>& G = grids[blockIdx.x];
    const int nlev = G.nlev, tid = threadIdx.x;
    // the lower levels run on the first wave
    const bool runB = nlev > 1 && tid < 64, runC = nlev > 2 && tid < 64;
    BatchLev<K, PA, 2, false> A(coef, G.g[0], uA);
    BatchLev<K, PB, 3, true> B(coef, G.g[1], uB);
    BatchLev<K, PC, 1, true> C(coef, G.g[2], uC);
    auto load = [&](auto& lev, int l) {
        lev.init_ghosts(G.g[l], G.old[l]);
#pragma unroll
        for (int q = 0; q < 2; ++q)
            if (lev.c[q] >= 0) {
                const int64_t e = lev.element(G.g[l], q);
                if constexpr (K::BASE) lev.cell[q].t0 = G.t0[l][e];
                else lev.cell[q].del = G.delta[l][e];
            }
    };
    T ref[2] = {T(0), T(0)};
#pragma unroll
    for (int q = 0; q < 2; ++q)
        if (A.c[q] >= 0) {
            const int64_t e = A.element(G.g[0], q);
            A.v[q] = G.u0[e];
            A.f[q] = G.f[e];
            ref[q] = G.old[0][e];
        }
    load(A, 0);
    if (runB) load(B, 1);
    if (runC) load(C, 2);
    if constexpr (K::BASE) {
        stage_base<PA, T8_NT>(G.g[0], pA, G.pt[0]);
        if (runB) stage_base<PB, 64>(G.g[1], pB, G.pt[1]);
        if (runC) stage_base<PC, 64>(G.g[2], pC, G.pt[2]);
    }
#pragma unroll
    for (int q = 0; q < 2; ++q)
        if (A.c[q] >= 0) oA[A.c[q]] = ref[q];
    __syncthreads();
    A.ghost_refs_at(oA);
    if constexpr (K::BASE) {
        base_cells<PA>(A, pA);
        if (runB) base_cells<PB>(B, pB);
        if (runC) base_cells<PC>(C, pC);
    }
    A.store_all();
    if (nlev == 1) {
        A.sweeps(ncoarse, true);
    } else {
        A.sweeps(nu1, false);
#pragma unroll
        for (int q = 0; q < 2; ++q)
            if (A.c[q] >= 0) dA[A.c[q]] = A.residual(q);
        __syncthreads();
        if (tid < 64) {
            T oldB[2] = {T(0), T(0)};
#pragma unroll
            for (int q = 0; q < 2; ++q)
                if (B.c[q] >= 0) {
                    oldB[q] = child_average<PA>(uA, B.i[q], B.j, B.z);
                    B.v[q] = oldB[q];
                    B.f[q] = child_average<PA>(dA, B.i[q], B.j, B.z);   // R d, then f^H
                }
            B.ghost_refs([&](int x, int y, int z) { return child_average<PA>(uA, x, y, z); });
            B.store_all();
#pragma unroll
            for (int q = 0; q < 2; ++q)
                if (B.c[q] >= 0) B.f[q] = B.residual(q);
            if (nlev == 2) {
                B.sweeps(ncoarse, true);
            } else {
                B.sweeps(nu1, false);
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    if (B.c[q] >= 0) dB[B.c[q]] = B.residual(q);
                wave_sync();
                T oldC[2] = {T(0), T(0)};
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    if (C.c[q] >= 0) {
                        oldC[q] = child_average<PB>(uB, C.i[q], C.j, C.z);
                        C.v[q] = oldC[q];
                        C.f[q] = child_average<PB>(dB, C.i[q], C.j, C.z);
                    }
                C.ghost_refs([&](int x, int y, int z) { return child_average<PB>(uB, x, y, z); });
                C.store_all();
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    if (C.c[q] >= 0) C.f[q] = C.residual(q);
                C.sweeps(ncoarse, true);
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    if (C.c[q] >= 0) uC[C.c[q]] = C.v[q] - oldC[q];
                wave_sync();
#pragma unroll
                for (int q = 0; q < 2; ++q)
                    if (B.c[q] >= 0) {
                        B.v[q] += prolong_at<PC>(uC, C.n0, C.n1, C.n2, B.i[q], B.j, B.z);
                        uB[B.c[q]] = B.v[q];
                    }
                wave_sync();
                B.sweeps(nu2, false);
            }
#pragma unroll
            for (int q = 0; q < 2; ++q)
                if (B.c[q] >= 0) uB[B.c[q]] = B.v[q] - oldB[q];
        }
        __syncthreads();
#pragma unroll
        for (int q = 0; q < 2; ++q)
            if (A.c[q] >= 0) {
                A.v[q] += prolong_at<PB>(uB, A.n0 >> 1, A.n1 >> 1, A.n2 >> 1, A.i[q], A.j, A.z);
                uA[A.c[q]] = A.v[q];
            }
        __syncthreads();
        A.sweeps(nu2, false);
    }
    // either ping-pong parity reads the result
#pragma unroll
    for (int q = 0; q < 2; ++q)
        if (A.c[q] >= 0) {
            const int64_t e = A.element(G.g[0], q);
            G.u0[e] = A.v[q];
            G.u1[e] = A.v[q];
        }
}

hipError_t launch_tail_batch(const TailGrid<double>* grids, int ngrids, const Coef& c, int nu1, int nu2, int ncoarse,
                             hipStream_t s) {
    if (ngrids <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_tail_batch<TailK>, dim3(ngrids), dim3(T8_NT), 0, s, grids, c, nu1, nu2, ncoarse);
    return hipGetLastError();
}

hipError_t launch_tail_batch(const TailGrid<float>* grids, int ngrids, const Coef& c, int nu1, int nu2, int ncoarse,
                             hipStream_t s) {
    if (ngrids <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_tail_batch<TailCorrK>, dim3(ngrids), dim3(T8_NT), 0, s, grids, c, nu1, nu2, ncoarse);
    return hipGetLastError();
}

// nlev levels from the one `a` describes, `next` the cells of the one below it
template <typename K>
static hipError_t tail_launch(const Tail<typename K::T>& a, int nlev, const int next[3], hipStream_t s) {
    const int64_t N = (int64_t)a.n[0] * a.n[1] * a.n[2];
    if (N < 1 || N > TAIL_CELLS || a.n[0] < 1 || a.n[1] < 1 || a.n[2] < 1) return hipErrorInvalidValue;
    if (nlev == 2) {
        for (int d = 0; d < 3; ++d)
            if (a.n[d] != 8 || next[d] != 4) return hipErrorInvalidValue;
        hipLaunchKernelGGL((k_tail8<K>), dim3(1), dim3(T8_NT), 0, s, a);
    } else if (nlev == 1) {
        if (N <= 64) hipLaunchKernelGGL((k_tail1<K, 64>), dim3(1), dim3(64), 0, s, a);
        else hipLaunchKernelGGL((k_tail1<K, 256>), dim3(1), dim3(256), 0, s, a);
    } else {
        return hipErrorInvalidValue;   // no periodic hierarchy has three levels of <= 512 cells
    }
    return hipGetLastError();
}

hipError_t launch_tail(const TailArgs& a, hipStream_t s) {
    Tail<double> t;
    for (int d = 0; d < 3; ++d) t.n[d] = a.n[0][d];
    t.h = a.h[0];
    t.delta = a.delta[0];
    t.delta_c = a.nlev > 1 ? a.delta[1] : nullptr;
    t.u = a.phi;
    t.f = a.f;
    t.pt = t.t0 = nullptr;
    t.sc = a.sc;
    t.pend = a.pend;
    t.c = a.c;
    t.nu1 = a.nu1; t.nu2 = a.nu2; t.ncoarse = a.ncoarse;
    return tail_launch<TailK>(t, a.nlev, a.n[1], s);
}

hipError_t launch_tail_corr(const TailCorrArgs& a, hipStream_t s) {
    Tail<float> t;
    for (int d = 0; d < 3; ++d) t.n[d] = a.n[0][d];
    t.h = a.h[0];
    t.delta = a.delta[0];
    t.delta_c = a.nlev > 1 ? a.delta[1] : nullptr;
    t.u = a.e;
    t.f = a.r;
    t.pt = a.pt;
    t.t0 = a.t0;
    t.sc = a.sc;
    t.pend = a.pend;
    t.c = a.c64;
    t.nu1 = a.nu1; t.nu2 = a.nu2; t.ncoarse = a.ncoarse;
    return tail_launch<TailCorrK>(t, a.nlev, a.n[1], s);
}

}  // namespace vmg
