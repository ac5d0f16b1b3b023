// Mass assignment: unit-mass particles to the density contrast on the periodic
// domain mesh or on a refinement region (Sec. VI: the mesh density comes from
// triangular-shaped-cloud assignment of the particles; cloud in cell is the
// next-lower-order member of the same family of shape functions).  A region is
// not periodic: each particle is taken from the periodic image that reaches
// it, and contributions outside it are dropped.
//
// Both schemes touch the particle's nearest cell and its 26 neighbours at most,
// so the grid is cut into bricks of 16^3 cells (8^3 on small grids, so that they
// fill the chip) and every particle belongs to the brick of its nearest cell:
//   1. k_count        particles per brick: each workgroup counts a contiguous
//                     range of particles in an LDS table with one counter per
//                     brick and adds the nonzero ones to one of the brick's
//                     global counters (SUB per brick); the brick of each particle
//                     is kept, or (region) the particles that reach it are listed;
//   2. k_scan_*       exclusive prefix sum of the counters;
//   3. k_place        the same ranges again: each nonzero (range, brick) count
//                     reserves a range of that brick's slots with one atomic,
//                     and the particle indices are written sorted by brick;
//   4. k_bin_assign   one workgroup per brick, or several where bricks are few
//                     and full (heaviest bricks first for the triangular-shaped
//                     cloud): the brick and a one-cell halo are accumulated in LDS
//                     and the region goes to the workspace;
//   5. k_gather       every cell sums the staged entries of the bricks that
//                     reach it (one; up to 8 on the outer layer of a brick, 27
//                     where bricks are one cell wide) and writes delta.
// Grids of more bricks than an LDS table holds count and place in chunks of 2048
// particles with an LDS hash table instead (k_bin).
// No global atomics touch the density.
// Masses are 64-bit fixed point (2^-40 of a particle per unit): every
// contribution is rounded once and all sums are integer, so the result does
// not depend on the order of particles or of atomics.
#include <algorithm>
#include <mutex>

#include "device_common.h"
#include "vmg_internal.h"

namespace vmg {
namespace {

constexpr double FIX_ONE = 1099511627776.0;           // 2^40
constexpr double FIX_INV = 1.0 / 1099511627776.0;     // 2^-40
constexpr int reg_edge(int B) { return B + 2; }        // brick of edge B + halo, LDS region edge
constexpr int reg_cells(int B) { return reg_edge(B) * reg_edge(B) * reg_edge(B); }
constexpr uint32_t NO_KEY = 0xffffffffu;

struct AGrid {
    int n0, n1, n2;          // cells
    int b0, b1, b2;          // bricks per axis
    int shift;               // log2 of the brick edge
    // refinement region (not periodic): cell size, corner of cell (0,0,0) and
    // n h + 2h per axis (offsets beyond it belong to the image below the corner)
    double h, cr[3], far[3];
};

// Periodic box: u = position in cells along an axis, in [0, n]; f = floor(u)
// unwrapped; the nearest cell is f mod n.
__device__ __forceinline__ double cells_of(double x, int n) { return (x - floor(x)) * (double)n; }

// Region: the offset from the corner taken modulo 1, moved below the corner
// when it lies beyond the region's far side plus two cells; in cells.
__device__ __forceinline__ double region_u(double x, double corner, double far, double h) {
    double d = x - corner;
    d -= floor(d);
    if (d > far) d -= 1.0;
    return d / h;
}

template <bool PER>
__device__ __forceinline__ double axis_u(const AGrid& g, int a, double x, int n) {
    if constexpr (PER)
        return cells_of(x, n);
    else
        return region_u(x, g.cr[a], g.far[a], g.h);
}

__device__ __forceinline__ bool finite3(double x, double y, double z) {
    return isfinite(x) && isfinite(y) && isfinite(z);
}

// Brick of the particle's nearest cell.  Region: a particle whose nearest cell
// is more than one cell outside reaches no cell of the region (NO_KEY); one
// cell outside, it goes to the brick on that face.
template <bool PER>
__device__ __forceinline__ uint32_t brick_key(const AGrid& g, double x, double y, double z) {
    const double f0 = floor(axis_u<PER>(g, 0, x, g.n0)), f1 = floor(axis_u<PER>(g, 1, y, g.n1)),
                 f2 = floor(axis_u<PER>(g, 2, z, g.n2));
    int c0, c1, c2;
    if constexpr (PER) {
        c0 = (int)f0;
        c1 = (int)f1;
        c2 = (int)f2;
        c0 -= c0 >= g.n0 ? g.n0 : 0;
        c1 -= c1 >= g.n1 ? g.n1 : 0;
        c2 -= c2 >= g.n2 ? g.n2 : 0;
    } else {
        // compared as doubles: far from a small region u can exceed the int range
        if (!(f0 >= -1.0 && f0 <= g.n0 && f1 >= -1.0 && f1 <= g.n1 && f2 >= -1.0 && f2 <= g.n2)) return NO_KEY;
        c0 = min(max((int)f0, 0), g.n0 - 1);
        c1 = min(max((int)f1, 0), g.n1 - 1);
        c2 = min(max((int)f2, 0), g.n2 - 1);
    }
    return ((uint32_t)(c2 >> g.shift) * g.b1 + (uint32_t)(c1 >> g.shift)) * g.b0 + (uint32_t)(c0 >> g.shift);
}

// round(a * b) as an integer, for 0 <= a * b < 2^51: the exact product plus
// 2^52 is rounded once (to nearest, ties to even) to a double whose low 52
// mantissa bits hold that integer.
__device__ __forceinline__ unsigned long long fix_round(double a, double b) {
    const double v = fma(a, b, 4503599627370496.0);
    return (unsigned long long)__double_as_longlong(v) & 0x000fffffffffffffull;
}

__global__ void __launch_bounds__(NT) k_fill_u32(uint32_t* __restrict__ p, int64_t n) {
    for (int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x; e < n; e += (int64_t)gridDim.x * NT) p[e] = 0u;
}

constexpr int ANT = 512;                              // threads of the brick accumulation
constexpr int SUB = 16;                               // counters per brick (range or chunk r uses r % SUB)
constexpr int CHUNK_PER_THREAD = 8;
constexpr int CHUNK = CHUNK_PER_THREAD * NT;          // particles per chunk
constexpr int TAB = 2 * CHUNK;                        // LDS hash table entries (load <= 1/2)
static_assert(TAB == 1 << 12, "the hash keeps the top 12 bits of the product");

// Counting and placing with a counter per brick in LDS.  Block b takes particles
// [b * per, (b + 1) * per).  Against the hashed chunks of k_bin a workgroup covers
// up to 8 times as many particles per table, so unordered particles cost that much
// fewer global atomics per brick, and no probing; ordered ones are counted a run of
// equal bricks at a time either way.  Whole calls: 200^3 particles in random order
// onto 200^3 cells (TSC) 800 -> 505 us, with 4096 ranges instead of 1024 788 us;
// 256^3 lattice-ordered ones: k_count 104 us (403 MB read at 4.5 TB/s), k_place 39 us
// against 49.  A region only keeps the particles that reach it: 7 M particles, 64^3
// cells of a 384^3 box: k_count 28 us, k_place 6 us against 32 and 13 us.
constexpr int CNT = 512;                              // threads
constexpr int CNT_BLOCKS = 1024;
constexpr int TAB_BRICKS = 1 << 14;                   // 64 KB of counters: two workgroups per CU

// Runs of equal keys among the lanes of a wave: whether this lane is the first of
// its run, that first lane, and (first lanes) the run's length.
struct Run {
    bool head;
    int first, len;
};
__device__ __forceinline__ Run key_run(uint32_t key) {
    const int lane = threadIdx.x & 63;
    const uint32_t prev = (uint32_t)__shfl_up((int)key, 1);
    Run r;
    r.head = lane == 0 || key != prev;
    const unsigned long long heads = __ballot(r.head), below = (2ull << lane) - 1ull;
    r.first = 63 - __clzll(heads & below);
    const unsigned long long after = heads & ~below;
    r.len = (after ? __ffsll(after) - 1 : 64) - lane;
    return r;
}

// PER: keys[p] receives particle p's brick.  Region: the block lists the particles
// of its range that reach the region (few, as a rule) at the start of its range of
// keys, and their number in listed[block].
template <bool PER>
__global__ void __launch_bounds__(CNT) k_count(AGrid g, const double* __restrict__ pos, int64_t np, int64_t per,
                                               uint32_t nb, uint32_t* __restrict__ counter,
                                               uint32_t* __restrict__ keys, uint32_t* __restrict__ listed) {
    extern __shared__ uint32_t tab[];
    __shared__ uint32_t n_listed;
    for (uint32_t e = threadIdx.x; e < nb; e += CNT) tab[e] = 0u;
    if (threadIdx.x == 0) n_listed = 0u;
    __syncthreads();
    const int64_t lo = blockIdx.x * per, hi = min(lo + per, np);
    constexpr int U = 4;                              // particles in flight per thread
    for (int64_t p0 = lo; p0 < hi; p0 += U * CNT) {
        double x[U], y[U], z[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t p = p0 + u * CNT + threadIdx.x;
            x[u] = y[u] = z[u] = __builtin_nan("");
            if (p < hi) {
                x[u] = pos[3 * p];
                y[u] = pos[3 * p + 1];
                z[u] = pos[3 * p + 2];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t p = p0 + u * CNT + threadIdx.x;
            uint32_t key = NO_KEY;
            if constexpr (PER) {
                if (finite3(x[u], y[u], z[u])) key = brick_key<PER>(g, x[u], y[u], z[u]);
                if (p < hi) keys[p] = key;
            } else {
                // most waves lie outside along z or y: one division, not three
                // (a coordinate that is not finite fails the comparisons)
                const double fz = floor(region_u(z[u], g.cr[2], g.far[2], g.h));
                if (!__any(fz >= -1.0 && fz <= g.n2)) continue;   // (uniform over the wave)
                const double fy = floor(region_u(y[u], g.cr[1], g.far[1], g.h));
                if (!__any(fy >= -1.0 && fy <= g.n1)) continue;
                if (finite3(x[u], y[u], z[u])) key = brick_key<PER>(g, x[u], y[u], z[u]);
                const unsigned long long in = __ballot(key != NO_KEY);
                if (in == 0) continue;
                const int lane = threadIdx.x & 63;
                uint32_t base = 0;
                if (lane == 0) base = atomicAdd(&n_listed, (uint32_t)__popcll(in));
                base = (uint32_t)__shfl((int)base, 0);
                if (key != NO_KEY) keys[lo + base + (uint32_t)__popcll(in & ((1ull << lane) - 1ull))] = (uint32_t)p;
            }
            const Run r = key_run(key);
            if (r.head && key != NO_KEY) atomicAdd(&tab[key], (uint32_t)r.len);
        }
    }
    __syncthreads();
    const uint32_t sub = blockIdx.x % SUB;
    for (uint32_t e = threadIdx.x; e < nb; e += CNT)
        if (tab[e]) atomicAdd(counter + (size_t)e * SUB + sub, tab[e]);
    if (!PER && threadIdx.x == 0) listed[blockIdx.x] = n_listed;
}

// The particles of this block's range again (PER: their keys; region: the listed
// ones): count, reserve, write.
template <bool PER>
__global__ void __launch_bounds__(CNT) k_place(AGrid g, const double* __restrict__ pos, int64_t np, int64_t per,
                                               uint32_t nb, uint32_t* __restrict__ cursor,
                                               const uint32_t* __restrict__ keys,
                                               const uint32_t* __restrict__ listed, uint32_t* __restrict__ idx) {
    extern __shared__ uint32_t tab[];
    for (uint32_t e = threadIdx.x; e < nb; e += CNT) tab[e] = 0u;
    __syncthreads();
    const int64_t lo = blockIdx.x * per, hi = PER ? min(lo + per, np) : lo + listed[blockIdx.x];
    if (!PER && lo == hi) return;
    constexpr int U = 4;
    auto load = [&](int64_t p0, uint32_t (&key)[U], uint32_t (&part)[U]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t p = p0 + u * CNT + threadIdx.x;
            key[u] = NO_KEY;
            part[u] = (uint32_t)p;
            if (p < hi) (PER ? key[u] : part[u]) = keys[p];
        }
        if constexpr (!PER) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t q = part[u];
                if (p0 + u * CNT + threadIdx.x < hi)
                    key[u] = brick_key<PER>(g, pos[3 * q], pos[3 * q + 1], pos[3 * q + 2]);
            }
        }
    };
    for (int64_t p0 = lo; p0 < hi; p0 += U * CNT) {
        uint32_t key[U], part[U];
        load(p0, key, part);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const Run r = key_run(key[u]);
            if (r.head && key[u] != NO_KEY) atomicAdd(&tab[key[u]], (uint32_t)r.len);
        }
    }
    __syncthreads();
    for (uint32_t e = threadIdx.x; e < nb; e += CNT)
        if (tab[e]) tab[e] = atomicAdd(cursor + (size_t)e * SUB + blockIdx.x % SUB, tab[e]);
    __syncthreads();
    for (int64_t p0 = lo; p0 < hi; p0 += U * CNT) {
        uint32_t key[U], part[U];
        load(p0, key, part);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const Run r = key_run(key[u]);
            uint32_t base = 0;
            if (r.head && key[u] != NO_KEY) base = atomicAdd(&tab[key[u]], (uint32_t)r.len);
            base = (uint32_t)__shfl((int)base, r.first);
            if (key[u] != NO_KEY) idx[base + (uint32_t)((threadIdx.x & 63) - r.first)] = part[u];
        }
    }
}

// MODE 0: add every chunk's per-brick counts to counter[] and store each
// particle's brick key.  MODE 1: reserve each chunk's range of every brick's
// slots from counter[] (the cursors) and write the particle indices there.
// Chunk ch counts into sub-counter ch % SUB of a brick, which spreads the
// global atomics of unordered particles over SUB addresses per brick.
// Bricks are found in the LDS table by linear probing from a multiplicative
// hash of the key.
template <int MODE, bool PER>
__global__ void __launch_bounds__(NT) k_bin(AGrid g, const double* __restrict__ pos, int64_t np,
                                            uint32_t* __restrict__ counter, uint32_t* __restrict__ keys,
                                            uint32_t* __restrict__ idx) {
    __shared__ uint32_t tkey[TAB], tcnt[TAB];
    __shared__ uint16_t used[CHUNK];                      // entries this chunk filled, in fill order
    __shared__ uint32_t n_used;
    for (int e = threadIdx.x; e < TAB; e += NT) {
        tkey[e] = NO_KEY;
        tcnt[e] = 0u;
    }
    if (threadIdx.x == 0) n_used = 0u;
    __syncthreads();
    const int64_t nchunk = (np + CHUNK - 1) / CHUNK;
    for (int64_t ch = blockIdx.x; ch < nchunk; ch += gridDim.x) {
        uint32_t key[CHUNK_PER_THREAD];
#pragma unroll
        for (int k = 0; k < CHUNK_PER_THREAD; ++k) {
            const int64_t p = ch * CHUNK + k * NT + threadIdx.x;
            key[k] = NO_KEY;
            if (p >= np) continue;
            if (MODE == 0) {
                const double x = pos[3 * p], y = pos[3 * p + 1], z = pos[3 * p + 2];
                if (finite3(x, y, z)) key[k] = brick_key<PER>(g, x, y, z);
                keys[p] = key[k];
            } else {
                key[k] = keys[p];
            }
        }
        // Lanes of a wavefront hold consecutive particles; a run of adjacent
        // lanes with one key is entered by its first lane, which reserves the
        // run's slots with one LDS atomic.
        const int lane = threadIdx.x & 63;
        const unsigned long long below = (2ull << lane) - 1ull;         // lanes 0..lane
        int hs[CHUNK_PER_THREAD];
        uint32_t loc[CHUNK_PER_THREAD];
#pragma unroll
        for (int k = 0; k < CHUNK_PER_THREAD; ++k) {
            const uint32_t prev = (uint32_t)__shfl_up((int)key[k], 1);
            const bool head = lane == 0 || key[k] != prev;
            const unsigned long long heads = __ballot(head);
            const int first = 63 - __clzll(heads & below);               // head of this lane's run
            const unsigned long long after = heads & ~below;
            const int len = (after ? __ffsll(after) - 1 : 64) - lane;    // run length, read by heads only
            int h = -1;
            uint32_t base = 0;
            if (head && key[k] != NO_KEY) {
                h = (int)((key[k] * 2654435761u) >> 20) & (TAB - 1);
                for (;;) {                                // at most CHUNK distinct keys: always a free entry
                    const uint32_t old = atomicCAS(&tkey[h], NO_KEY, key[k]);
                    if (old == NO_KEY) {
                        used[atomicAdd(&n_used, 1u)] = (uint16_t)h;
                        break;
                    }
                    if (old == key[k]) break;
                    h = (h + 1) & (TAB - 1);
                }
                base = atomicAdd(&tcnt[h], (uint32_t)len);
            }
            hs[k] = __shfl(h, first);
            loc[k] = (uint32_t)__shfl((int)base, first) + (uint32_t)(lane - first);
            if (key[k] == NO_KEY) hs[k] = -1;
        }
        __syncthreads();
        const uint32_t sub = (uint32_t)(ch % SUB);
        const int nu = (int)n_used;
        for (int u = threadIdx.x; u < nu; u += NT) {
            const int e = used[u];
            const uint32_t k = tkey[e];
            if (MODE == 0)
                atomicAdd(counter + (size_t)k * SUB + sub, tcnt[e]);
            else
                tcnt[e] = atomicAdd(counter + (size_t)k * SUB + sub, tcnt[e]);   // this chunk's first slot
        }
        if (MODE == 1) {
            __syncthreads();
#pragma unroll
            for (int k = 0; k < CHUNK_PER_THREAD; ++k)
                if (hs[k] >= 0) idx[tcnt[hs[k]] + loc[k]] = (uint32_t)(ch * CHUNK + k * NT + threadIdx.x);
        }
        __syncthreads();
        // empty the filled entries for the next chunk
        for (int u = threadIdx.x; u < nu; u += NT) {
            const int e = used[u];
            tkey[e] = NO_KEY;
            tcnt[e] = 0u;
        }
        __syncthreads();
        if (threadIdx.x == 0) n_used = 0u;
        __syncthreads();
    }
}

// Exclusive prefix sum of the nc counters into start[0..nc] and cursor[0..nc),
// in three launches: per-block sums of SCAN_TILE counters, an exclusive scan
// of those sums in one block, and block-local scans offset by them.
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* part, uint32_t* total) {
    const int t = threadIdx.x;
    part[t] = v;
    __syncthreads();
    for (int off = 1; off < NT; off <<= 1) {                 // inclusive Hillis-Steele scan
        const uint32_t u = t >= off ? part[t - off] : 0u;
        __syncthreads();
        part[t] += u;
        __syncthreads();
    }
    const uint32_t incl = part[t];
    *total = part[NT - 1];
    __syncthreads();
    return incl - v;
}

constexpr int SCAN_PER_THREAD = 16;
constexpr int SCAN_TILE = SCAN_PER_THREAD * NT;

__global__ void __launch_bounds__(NT) k_scan_sums(const uint32_t* __restrict__ count, int64_t nc,
                                                  uint32_t* __restrict__ sums) {
    __shared__ uint32_t part[NT];
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_PER_THREAD;
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < SCAN_PER_THREAD; ++k) s += base + k < nc ? count[base + k] : 0u;
    uint32_t total;
    block_exclusive_scan(s, part, &total);
    if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

// One block: exclusive scan of the m tile sums in place (contiguous runs per thread).
__global__ void __launch_bounds__(NT) k_scan_top(uint32_t* __restrict__ sums, int64_t m) {
    __shared__ uint32_t part[NT];
    const int64_t per = (m + NT - 1) / NT;
    const int64_t lo = threadIdx.x * per, hi = lo + per < m ? lo + per : m;
    uint32_t s = 0;
    for (int64_t b = lo; b < hi; ++b) s += sums[b];
    uint32_t total;
    uint32_t run = block_exclusive_scan(s, part, &total);
    for (int64_t b = lo; b < hi; ++b) {
        const uint32_t v = sums[b];
        sums[b] = run;
        run += v;
    }
}

__global__ void __launch_bounds__(NT) k_scan_tiles(const uint32_t* __restrict__ count, int64_t nc,
                                                   const uint32_t* __restrict__ sums, uint32_t* __restrict__ start,
                                                   uint32_t* __restrict__ cursor) {
    __shared__ uint32_t part[NT];
    const int64_t base = (int64_t)blockIdx.x * SCAN_TILE + (int64_t)threadIdx.x * SCAN_PER_THREAD;
    uint32_t v[SCAN_PER_THREAD];
    uint32_t s = 0;
#pragma unroll
    for (int k = 0; k < SCAN_PER_THREAD; ++k) {
        v[k] = base + k < nc ? count[base + k] : 0u;
        s += v[k];
    }
    uint32_t total;
    uint32_t run = sums[blockIdx.x] + block_exclusive_scan(s, part, &total);
#pragma unroll
    for (int k = 0; k < SCAN_PER_THREAD; ++k) {
        if (base + k < nc) {
            start[base + k] = run;
            cursor[base + k] = run;
        }
        run += v[k];
    }
    if (base + SCAN_PER_THREAD >= nc && base < nc) start[nc] = run;    // the thread holding the last counter
}

// The same in one launch of one block, for up to SCAN_ONE counters (a launch costs
// more than one CU's scan of them): thread t takes `per` consecutive counters (a
// multiple of 4), read twice.
constexpr int SCAN_NT = 1024;
constexpr int64_t SCAN_ONE = 1 << 14;
__global__ void __launch_bounds__(SCAN_NT) k_scan_one(const uint32_t* __restrict__ count, int nc, int per,
                                                      uint32_t* __restrict__ start, uint32_t* __restrict__ cursor) {
    __shared__ uint32_t wsum[SCAN_NT / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, lo = threadIdx.x * per;
    const uint4* c4 = reinterpret_cast<const uint4*>(count);   // nc is a multiple of SUB
    uint32_t sum = 0;
#pragma unroll 4
    for (int k = 0; k < per; k += 4)
        if (lo + k < nc) {
            const uint4 v = c4[(lo + k) >> 2];
            sum += v.x + v.y + v.z + v.w;
        }
    uint32_t incl = sum;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t u = (uint32_t)__shfl_up((int)incl, o);
        incl += lane >= o ? u : 0u;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    uint32_t run = incl - sum;
#pragma unroll
    for (int q = 0; q < SCAN_NT / 64; ++q) run += q < wave ? wsum[q] : 0u;
#pragma unroll 4
    for (int k = 0; k < per; k += 4)
        if (lo + k < nc) {
            const uint4 v = c4[(lo + k) >> 2];
            uint4 o;
            o.x = run;
            o.y = o.x + v.x;
            o.z = o.y + v.y;
            o.w = o.z + v.z;
            run = o.w + v.w;
            reinterpret_cast<uint4*>(start)[(lo + k) >> 2] = o;
            reinterpret_cast<uint4*>(cursor)[(lo + k) >> 2] = o;
        }
    if (lo < nc && lo + per >= nc) start[nc] = run;
}
static_assert(SUB % 4 == 0, "counters come in fours");

// Brick-local LDS index of a cell whose brick-local coordinates are l0, l1, l2
// in [-1, B].
template <int B>
__device__ __forceinline__ int reg_index(int l0, int l1, int l2) {
    return ((l2 + 1) * reg_edge(B) + (l1 + 1)) * reg_edge(B) + (l0 + 1);
}

template <int B>
__device__ __forceinline__ bool in_reg(int l) { return (unsigned)(l + 1) <= (unsigned)(B + 1); }

// Per-axis local cells (brick-local coordinate of the first stencil cell) and
// weights.  CIC: weights 1 - t, t on cells floor(u - 1/2) and the next; TSC:
// nearest cell c, d = u - (c + 1/2), weights (1/2 - d)^2/2, 3/4 - d^2,
// (1/2 + d)^2/2 on cells c - 1, c, c + 1.  `org` is the brick's first cell.
template <int M, bool PER>
__device__ __forceinline__ int axis_local(double u, int n, int org, double (&w)[M]) {
    const double f = floor(u);
    int c = (int)f;
    if constexpr (PER) c -= c >= n ? n : 0;               // nearest cell, in this brick (region: may be -1 or n)
    if constexpr (M == 2) {
        const double g = floor(u - 0.5);                  // f - 1 or f
        const double t = (u - 0.5) - g;
        w[0] = 1.0 - t;
        w[1] = t;
        return c - org + (int)(g - f);
    } else {
        const double d = u - (f + 0.5);
        const double a = 0.5 - d, b = 0.5 + d;
        w[0] = 0.5 * (a * a);
        w[1] = 0.75 - d * d;
        w[2] = 0.5 * (b * b);
        return c - org - 1;
    }
}

// Bricks in order of decreasing particle count (64 buckets of 128 particles;
// one block), so the heaviest bricks start first and do not trail the launch
// (used for the triangular-shaped cloud, whose per-particle work makes the
// imbalance worth the extra launch).
constexpr int ORD_NT = 1024;
__global__ void __launch_bounds__(ORD_NT) k_brick_order(const uint32_t* __restrict__ start, int64_t nb,
                                                        uint32_t* __restrict__ order) {
    __shared__ uint32_t hist[64];
    if (threadIdx.x < 64) hist[threadIdx.x] = 0u;
    __syncthreads();
    for (int64_t b = threadIdx.x; b < nb; b += ORD_NT) {
        const uint32_t cnt = start[(b + 1) * SUB] - start[b * SUB];
        atomicAdd(&hist[63 - min(cnt >> 7, 63u)], 1u);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t run = 0;
        for (int k = 0; k < 64; ++k) {
            const uint32_t v = hist[k];
            hist[k] = run;
            run += v;
        }
    }
    __syncthreads();
    for (int64_t b = threadIdx.x; b < nb; b += ORD_NT) {
        const uint32_t cnt = start[(b + 1) * SUB] - start[b * SUB];
        order[atomicAdd(&hist[63 - min(cnt >> 7, 63u)], 1u)] = (uint32_t)b;
    }
}

// SPLIT: `split` workgroups share a brick's particles and add their regions to the
// zeroed staging area; else a workgroup writes its brick's region.
template <int M, bool PER, int B, bool SPLIT>
__global__ void __launch_bounds__(ANT) k_bin_assign(AGrid g, const double* __restrict__ pos,
                                                   const uint32_t* __restrict__ start,
                                                   const uint32_t* __restrict__ idx,
                                                   const uint32_t* __restrict__ order, int split,
                                                   unsigned long long* __restrict__ stage) {
    constexpr int REGN = reg_cells(B);
    __shared__ unsigned long long acc[REGN];
    const int item = SPLIT ? (int)blockIdx.x / split : (int)blockIdx.x;
    const int key = order ? (int)order[item] : item;
    uint32_t lo = start[(size_t)key * SUB], hi = start[(size_t)(key + 1) * SUB];
    if (SPLIT) {
        const uint32_t s = blockIdx.x % split, n = hi - lo;
        hi = lo + (uint32_t)((uint64_t)n * (s + 1) / split);
        lo += (uint32_t)((uint64_t)n * s / split);
        if (lo == hi) return;
    }
    const int bx = key % g.b0, by = (key / g.b0) % g.b1, bz = key / (g.b0 * g.b1);
    const int o0 = bx * B, o1 = by * B, o2 = bz * B;
    for (int e = threadIdx.x; e < REGN; e += ANT) acc[e] = 0ull;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const int rx = lane % M, ry = (lane >> 4) % M;
    for (uint32_t t = lo + threadIdx.x; t < hi; t += ANT) {
        const int64_t p = idx[t];
        const double x = pos[3 * p], y = pos[3 * p + 1], z = pos[3 * p + 2];
        double wx[M], wy[M], wz[M];
        const int l0 = axis_local<M, PER>(axis_u<PER>(g, 0, x, g.n0), g.n0, o0, wx);
        const int l1 = axis_local<M, PER>(axis_u<PER>(g, 1, y, g.n1), g.n1, o1, wy);
        const int l2 = axis_local<M, PER>(axis_u<PER>(g, 2, z, g.n2), g.n2, o2, wz);
        // rotate the x and y stencil order by lane so that neighbouring lanes
        // (often the same nearest cell) add to different cells in one instruction
        double wxr[M], wyr[M];
        int oxr[M], oyr[M];
#pragma unroll
        for (int c = 0; c < M; ++c) {
            const int sx = c + rx >= M ? c + rx - M : c + rx;
            const int sy = c + ry >= M ? c + ry - M : c + ry;
            wxr[c] = wx[0];
            wyr[c] = wy[0];
#pragma unroll
            for (int q = 1; q < M; ++q) {
                wxr[c] = sx == q ? wx[q] : wxr[c];
                wyr[c] = sy == q ? wy[q] : wyr[c];
            }
            oxr[c] = sx;
            oyr[c] = sy;
        }
#pragma unroll
        for (int a = 0; a < M; ++a) {
#pragma unroll
            for (int b = 0; b < M; ++b) {
                const double wyz = wz[a] * wyr[b] * FIX_ONE;
                const int r = reg_index<B>(l0, l1 + oyr[b], l2 + a);
#pragma unroll
                for (int c = 0; c < M; ++c) {
                    // region: a stencil cell beyond the LDS halo lies outside
                    // the region; its contribution is dropped
                    if (!PER && !(in_reg<B>(l0 + oxr[c]) && in_reg<B>(l1 + oyr[b]) && in_reg<B>(l2 + a))) continue;
                    atomicAdd(&acc[r + oxr[c]], fix_round(wxr[c], wyz));
                }
            }
        }
    }
    __syncthreads();
    unsigned long long* st = stage + (size_t)key * REGN;
    for (int e = threadIdx.x; e < REGN; e += ANT) {
        if (!SPLIT) st[e] = acc[e];
        else if (acc[e]) atomicAdd(st + e, acc[e]);
    }
}

__global__ void __launch_bounds__(NT) k_fill_u64(unsigned long long* __restrict__ p, int64_t n) {
    for (int64_t e = (int64_t)blockIdx.x * NT + threadIdx.x; e < n; e += (int64_t)gridDim.x * NT) p[e] = 0ull;
}

// The (brick, brick-local coordinate) pairs along one axis whose LDS region
// entries land on cell i: the cell's own brick, and for the first (last) cell
// of a brick the right (left) halo entry of the previous (next) brick, with
// periodic wrap (a region has no brick before its first or after its last);
// returns how many (1 to 3).
template <int B>
__device__ __forceinline__ int axis_sources(int i, int n, int nbrick, bool periodic, int (&b)[3], int (&l)[3]) {
    const int bi = i / B, li = i - bi * B, w = min(B, n - bi * B);
    int m = 0;
    b[m] = bi;
    l[m++] = li;
    if (li == 0 && (periodic || bi > 0)) {
        const int bp = bi == 0 ? nbrick - 1 : bi - 1;
        b[m] = bp;
        l[m++] = min(B, n - bp * B);
    }
    if (li == w - 1 && (periodic || bi < nbrick - 1)) {
        b[m] = bi == nbrick - 1 ? 0 : bi + 1;
        l[m++] = -1;
    }
    return m;
}

// Every cell: the sum of the staged region entries of the bricks that reach it
// (its own brick's entry, plus halo entries of neighbours for outer-layer
// cells), converted to delta = q * scale - 1.  A block writes 64 columns of one
// plane of a row of bricks (blockIdx.x = brick row and column tile, blockIdx.y =
// k), so the staged plane of each brick is read through whole lines; a thread
// takes B/4 rows of its column (that many loads in flight, its sources found
// once).  256^3 cells: 85 us (325 MB at 3.8 TB/s); with a block per row of cells,
// which read every line of the staged planes twice and found its sources for one
// cell per thread, 139 us.
constexpr int GCOLS = 64, GROUPS = NT / GCOLS;
template <int B>
__global__ void __launch_bounds__(NT) k_gather(AGrid g, bool periodic, const unsigned long long* __restrict__ stage,
                                               double scale, double* __restrict__ d) {
    constexpr int REG = reg_edge(B), REGN = reg_cells(B), RT = B / GROUPS;
    const int tiles = (g.n0 + GCOLS - 1) / GCOLS;
    const int by = blockIdx.x / tiles, k = blockIdx.y;
    const int i = (blockIdx.x % tiles) * GCOLS + threadIdx.x % GCOLS;
    const int r0 = threadIdx.x / GCOLS * RT;          // first of this thread's rows of the brick row
    const int w = min(B, g.n1 - by * B);              // rows there are
    if (i >= g.n0 || r0 >= w) return;
    int b0[3], l0[3], b2[3], l2[3];
    const int m0 = axis_sources<B>(i, g.n0, g.b0, periodic, b0, l0);
    const int m2 = axis_sources<B>(k, g.n2, g.b2, periodic, b2, l2);
    unsigned long long q[RT];
#pragma unroll
    for (int r = 0; r < RT; ++r) q[r] = 0ull;
    for (int c = 0; c < m2; ++c)
        for (int a = 0; a < m0; ++a) {
            const unsigned long long* plane =
                stage + (((size_t)b2[c] * g.b1) * g.b0 + b0[a]) * REGN + reg_index<B>(l0[a], 0, l2[c]);
            const unsigned long long* own = plane + (size_t)by * g.b0 * REGN + r0 * REG;
#pragma unroll
            for (int r = 0; r < RT; ++r)
                if (r0 + r < w) q[r] += own[r * REG];
            // the first and last rows also take halo entries of the brick rows around
#pragma unroll
            for (int r = 0; r < RT; ++r) {
                if (r0 + r >= w || (r0 + r != 0 && r0 + r != w - 1)) continue;
                int b1[3], l1[3];
                const int m1 = axis_sources<B>(by * B + r0 + r, g.n1, g.b1, periodic, b1, l1);
                for (int b = 1; b < m1; ++b) q[r] += plane[(size_t)b1[b] * g.b0 * REGN + l1[b] * REG];
            }
        }
    double* out = d + ((int64_t)k * g.n1 + by * B + r0) * g.n0 + i;
#pragma unroll
    for (int r = 0; r < RT; ++r)
        if (r0 + r < w) out[(int64_t)r * g.n0] = (double)q[r] * scale - 1.0;
}

inline int64_t align256(int64_t b) { return (b + 255) & ~(int64_t)255; }

}  // namespace

static int64_t bricks_of(int n0, int n1, int n2, int B) {
    return (int64_t)((n0 + B - 1) / B) * ((n1 + B - 1) / B) * ((n2 + B - 1) / B);
}

int64_t mass_assign_bricks(int n0, int n1, int n2) { return bricks_of(n0, n1, n2, 16); }

static int64_t workspace_of(int64_t np, int n0, int n1, int n2, int B) {
    const int64_t nb = bricks_of(n0, n1, n2, B), nc = nb * SUB;
    return 2 * align256(nc * 4) + align256((nc + 1) * 4) + align256((nc + SCAN_TILE - 1) / SCAN_TILE * 4) +
           2 * align256(np * 4) + align256(nb * reg_cells(B) * 8) + align256(nb * 4);
}

// Grids of fewer than 128 bricks of 16^3 cells are cut into 8^3 ones where the
// workspace has room for their wider halos: 262144 particles onto 64^3 cells (CIC)
// take 34 us a call so, 51 us with 64 workgroups on 16^3 bricks, whose accumulation
// alone was 17 us against 8.  Above that the eightfold number of bricks costs
// unordered particles more global counter updates than the shorter workgroups save:
// 152 x 76 x 128 cells (400 bricks), 4.7 M particles in random order, TSC: 207 us,
// 352 us on 8^3 bricks; 96^3 cells, 1 M particles: 83 us against 126 us (ordered: 64
// against 66 us).
constexpr int64_t SMALL_BRICKS = 128;
constexpr int64_t SPLIT_BRICKS = 1024;
static bool small_grid(int n0, int n1, int n2) { return bricks_of(n0, n1, n2, 16) < SMALL_BRICKS; }

int64_t mass_assign_workspace_min(int64_t np, int n0, int n1, int n2) { return workspace_of(np, n0, n1, n2, 16); }

int64_t mass_assign_workspace(int64_t np, int n0, int n1, int n2) {
    const int64_t need = workspace_of(np, n0, n1, n2, 16);
    return small_grid(n0, n1, n2) ? std::max(need, workspace_of(np, n0, n1, n2, 8)) : need;
}

// Workspace of the allocation-free mass assignment: a file-scope device array
// that every GPU the library runs on holds until the process ends.  Host code
// must not use the array's name as an address (it is a host-side stand-in);
// noalloc_scratch() returns the device address, looked up once per device.
static __device__ __align__(256) unsigned char scratch[NOALLOC_SCRATCH_BYTES];

namespace {
std::mutex g_scratch_mu;
void* g_scratch_ptr[NOALLOC_MAX_DEVICES] = {};
}  // namespace

hipError_t noalloc_scratch(void** ptr) {
    *ptr = nullptr;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= NOALLOC_MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p || reinterpret_cast<uintptr_t>(p) % 256 != 0) return hipErrorInvalidValue;
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return hipSuccess;
}

template <int M, bool PER, int B>
static void assign_launch(const AGrid& g, const double* pos, const uint32_t* start, const uint32_t* idx,
                          const uint32_t* order, int split, int64_t nb, unsigned long long* stage, hipStream_t s) {
    if (split > 1) {
        hipLaunchKernelGGL(k_fill_u64, dim3(grid_for(nb * reg_cells(B), 2048)), dim3(NT), 0, s, stage,
                           nb * reg_cells(B));
        hipLaunchKernelGGL((k_bin_assign<M, PER, B, true>), dim3((unsigned)(nb * split)), dim3(ANT), 0, s, g, pos,
                           start, idx, order, split, stage);
    } else {
        hipLaunchKernelGGL((k_bin_assign<M, PER, B, false>), dim3((unsigned)nb), dim3(ANT), 0, s, g, pos, start, idx,
                           order, split, stage);
    }
}

hipError_t launch_mass_assign(const double* pos, int64_t np, int n0, int n1, int n2, int scheme, bool periodic,
                              double h, const double* corner, double mean_count, void* work, int64_t work_bytes,
                              double* delta, hipStream_t s) {
    const int B = small_grid(n0, n1, n2) && work_bytes >= workspace_of(np, n0, n1, n2, 8) ? 8 : 16;
    AGrid g{n0, n1, n2, (n0 + B - 1) / B, (n1 + B - 1) / B, (n2 + B - 1) / B, B == 8 ? 3 : 4, h, {0, 0, 0},
            {0, 0, 0}};
    const int nn[3] = {n0, n1, n2};
    if (!periodic)
        for (int a = 0; a < 3; ++a) {
            g.cr[a] = corner[a];
            g.far[a] = nn[a] * h + 2.0 * h;
        }
    const int64_t nb = (int64_t)g.b0 * g.b1 * g.b2, nc = nb * SUB;
    char* w = static_cast<char*>(work);
    uint32_t* count = reinterpret_cast<uint32_t*>(w);
    w += align256(nc * 4);
    uint32_t* cursor = reinterpret_cast<uint32_t*>(w);
    w += align256(nc * 4);
    uint32_t* start = reinterpret_cast<uint32_t*>(w);
    w += align256((nc + 1) * 4);
    uint32_t* sums = reinterpret_cast<uint32_t*>(w);
    const int64_t ntile = (nc + SCAN_TILE - 1) / SCAN_TILE;
    w += align256(ntile * 4);
    uint32_t* keys = reinterpret_cast<uint32_t*>(w);
    w += align256(np * 4);
    uint32_t* idx = reinterpret_cast<uint32_t*>(w);
    w += align256(np * 4);
    unsigned long long* stage = reinterpret_cast<unsigned long long*>(w);
    w += align256(nb * reg_cells(B) * 8);
    uint32_t* order = reinterpret_cast<uint32_t*>(w);
    const double scale = FIX_INV / mean_count;
    hipLaunchKernelGGL(k_fill_u32, dim3(grid_for(nc)), dim3(NT), 0, s, count, nc);
    const bool table = nb <= TAB_BRICKS;
    const int chunks = grid_for((np + CHUNK - 1) / CHUNK * NT, 8192);
    // one range per block, whole iterations of four particles per thread
    const int64_t iter = 4 * CNT, blocks = std::min<int64_t>(CNT_BLOCKS, (np + iter - 1) / iter);
    const int64_t per = ((np + blocks - 1) / blocks + iter - 1) / iter * iter;
    const dim3 ranges((unsigned)((np + per - 1) / per));
    const size_t lds = (size_t)nb * 4;
    // a region's list lengths wait in the staging area, which is written after them
    uint32_t* listed = reinterpret_cast<uint32_t*>(stage);
    static_assert(CNT_BLOCKS * 4 <= reg_cells(8) * 8, "room for the list lengths");
    if (table && periodic)
        hipLaunchKernelGGL(k_count<true>, ranges, dim3(CNT), lds, s, g, pos, np, per, (uint32_t)nb, count, keys, listed);
    else if (table)
        hipLaunchKernelGGL(k_count<false>, ranges, dim3(CNT), lds, s, g, pos, np, per, (uint32_t)nb, count, keys, listed);
    else if (periodic)
        hipLaunchKernelGGL((k_bin<0, true>), dim3(chunks), dim3(NT), 0, s, g, pos, np, count, keys, idx);
    else
        hipLaunchKernelGGL((k_bin<0, false>), dim3(chunks), dim3(NT), 0, s, g, pos, np, count, keys, idx);
    if (nc <= SCAN_ONE) {
        const int per4 = (int)((nc + 4 * SCAN_NT - 1) / (4 * SCAN_NT)) * 4;
        hipLaunchKernelGGL(k_scan_one, dim3(1), dim3(SCAN_NT), 0, s, count, (int)nc, per4, start, cursor);
    } else {
        hipLaunchKernelGGL(k_scan_sums, dim3((unsigned)ntile), dim3(NT), 0, s, count, nc, sums);
        hipLaunchKernelGGL(k_scan_top, dim3(1), dim3(NT), 0, s, sums, ntile);
        hipLaunchKernelGGL(k_scan_tiles, dim3((unsigned)ntile), dim3(NT), 0, s, count, nc, sums, start, cursor);
    }
    if (table && periodic)
        hipLaunchKernelGGL(k_place<true>, ranges, dim3(CNT), lds, s, g, pos, np, per, (uint32_t)nb, cursor, keys,
                           listed, idx);
    else if (table)
        hipLaunchKernelGGL(k_place<false>, ranges, dim3(CNT), lds, s, g, pos, np, per, (uint32_t)nb, cursor, keys,
                           listed, idx);
    else
        hipLaunchKernelGGL((k_bin<1, true>), dim3(chunks), dim3(NT), 0, s, g, pos, np, cursor, keys, idx);
    // workgroups per brick: doubled while there are fewer than four per CU (so fewer
    // than eight in the end) and each keeps at least 2048 particles of a brick of
    // average content (4.3 M particles in random order onto 32 x 131 x 28
    // cells, CIC: 172 us a call, 457 us with one workgroup per 16^3 brick; the 400
    // bricks above with ordered particles: 149 us, 222 us with one workgroup each)
    const double content = mean_count * (double)n0 * n1 * n2 / (double)nb;
    int split = 1;
    while (nb * split < SPLIT_BRICKS && content >= 4096.0 * split) split *= 2;
    // (an order only matters where bricks queue for the CUs)
    if (scheme == 2 && nb > SMALL_BRICKS)
        hipLaunchKernelGGL(k_brick_order, dim3(1), dim3(ORD_NT), 0, s, start, nb, order);
    else
        order = nullptr;
#define VMG_ASSIGN(M, PER)                                                                                  \
    do {                                                                                                    \
        if (B == 8) assign_launch<M, PER, 8>(g, pos, start, idx, order, split, nb, stage, s);               \
        else assign_launch<M, PER, 16>(g, pos, start, idx, order, split, nb, stage, s);                     \
    } while (0)
    if (scheme == 1 && periodic) VMG_ASSIGN(2, true);
    else if (scheme == 1) VMG_ASSIGN(2, false);
    else if (periodic) VMG_ASSIGN(3, true);
    else VMG_ASSIGN(3, false);
#undef VMG_ASSIGN
    const dim3 gather((unsigned)(g.b1 * ((n0 + GCOLS - 1) / GCOLS)), (unsigned)n2);
    if (B == 8) hipLaunchKernelGGL(k_gather<8>, gather, dim3(NT), 0, s, g, periodic, stage, scale, delta);
    else hipLaunchKernelGGL(k_gather<16>, gather, dim3(NT), 0, s, g, periodic, stage, scale, delta);
    return hipGetLastError();
}

}  // namespace vmg
