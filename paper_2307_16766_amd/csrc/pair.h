// pair.h -- two time steps per pass over HBM (gfx950).
//
// A single step (k_step) reads and writes every population once: on grids that do not stay in the
// caches it runs at the HBM rate, 2 q s bytes per node and step.  Here one pass takes the bulk from
// level n to level n + 2: a work-group owns an x tile of `wo` output columns and marches through a
// segment of rows; the level-(n+1) rows between the two steps live in LDS only.
//
//   - Thread group 0 (NT threads, one column each) pulls row r of level n + 1 from A (loads of row
//     r + 1 are issued before the barriers of row r, a whole row ahead of their use) and collides.
//   - Thread group 1 (NT threads) pulls output row r - M of level n + 2 from the LDS rows, collides
//     and stores it with non-temporal stores.
//   - LDS: population i of row r is read once, for output row r + c_iy, so it is kept for
//     M + 1 + c_iy rows only (a ring per population): (M + 1) q values per column on average 4 q
//     for M = 3 instead of (2 M + 1) q.  Writer and reader of a ring meet between two barriers per
//     row (write, barrier, read, barrier); both groups collide outside them, at the same time.
//   - The tile's columns include M halo columns on each side, recomputed by the neighbouring tile, and
//     a segment starts 2 M rows early; wo is a multiple of 64 bytes, so no 64-byte block of a row is
//     written by two work-groups.
//
// Boundary layers of level n + 1 are inputs of the second step: they come from band buffers (C), which
// k_bnd fills before the pass (the sides' solve n -> n + 1 writes the layers there, further
// work-groups the bulk nodes next to them), and from which a second k_bnd launch takes the sides
// from n + 1 to n + 2.  A band holds the BW = 3 M + 3 nodes next to a side, enough for every pull of
// the boundary solve (x_f - M - 2 - M is the innermost node it reads).  Layers of Dirichlet sides
// are the same at every level and are read from A itself.
// What bounds it: memory.  A pass over a periodic 4096 x 2048 takes 493 us in FP32 D2Q37, 482 without the
// collisions and 400 without the global loads and stores (about 680 vector instructions per node and
// step beside the LDS rings); in FP64 935, 940 and 645; D2Q17 FP64 on 1950 x 1950 212, 206 and 94.  Halo
// columns and rows cost little traffic: of the algorithmic bytes of one single step HBM reads 1.08 and
// writes 1.05 times in FP32, 1.07 and 1.01 in FP64 (counters, D2Q37 4096 x 2048 with open sides).
// Measured per step against the single-step kernel: D2Q37 4096 x 2048 FP64 periodic 820 -> 468 us, FP32
// with Dirichlet / LODI-RELAX sides 417 -> 277 us; D2Q17 FP64 1950 x 1950 186 -> 106 us; D2Q9 FP32 2048 x 2048
// 58 -> 26 us.  Requesting rows two or three ahead changed nothing (the
// loads are not the bound), tiles of half the columns with two work-groups per CU are slower (more
// halo), unaligned output tiles too (partial lines).
#pragma once

#include <utility>

#include "kernels.h"

namespace lbm {

// f(integral_constant<int, 0>) .. f(integral_constant<int, N - 1>): an index usable in constant expressions
template <int N, typename F> __device__ __forceinline__ void each(F&& f) {
    [&]<int... I>(std::integer_sequence<int, I...>) { (f(std::integral_constant<int, I>{}), ...); }(std::make_integer_sequence<int, N>{});
}

template <int Q> constexpr int BW = 3 * Lat<Q>::M + 3;       // band width (nodes from the side inward)
template <int Q> constexpr int CPX = 2 * BW<Q> <= 16 ? 16 : 32;   // row pitch of the x-band buffer (both sides)

// ------------------------------------------------------------------ LDS rings
template <int Q> constexpr int ring_len(int c) { return Lat<Q>::M + 1 + c; }
template <int Q> constexpr int ring_rank(int i) {            // populations before i with the same c_y
    int n = 0;
    for (int j = 0; j < i; ++j) n += cy<Q>(j) == cy<Q>(i);
    return n;
}
template <int Q> constexpr int ring_base(int c) {            // slots of the groups before c
    int n = 0;
    for (int j = 0; j < Q; ++j) n += cy<Q>(j) < c ? ring_len<Q>(cy<Q>(j)) : 0;
    return n;
}
template <int Q> constexpr int ring_slots() { return ring_base<Q>(Lat<Q>::M + 1); }
// first slot of population i's ring
template <int Q> constexpr int ring_of(int i) { return ring_base<Q>(cy<Q>(i)) + ring_rank<Q>(i) * ring_len<Q>(cy<Q>(i)); }

// columns (threads per group) of a work-group: the largest multiple of 64 up to 256 whose rings fit
// the CU's 160 KB of LDS
template <int Q, typename T> constexpr int pair_cols() {
    int n = 256;
    while ((size_t)ring_slots<Q>() * n * sizeof(T) > 160 * 1024) n -= 64;
    return n;
}

template <typename T> struct PairArgs {
    int nx, ny, x0, x1, y0, y1;    // bulk node range (inclusive)
    unsigned long long pitch;
    float omega_f;
    double omega_d;
    int wo, ntx, nseg;             // output columns per tile, tiles per row, row segments
    View<T> lay[4];                // layers of level n + 1 of the sides (unused where periodic)
};

// barrier ordering LDS only: the global loads and stores of the groups stay in flight across it
__device__ __forceinline__ void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// ring slots: per c_y the slot that the present row writes; the next one is the oldest
template <int Q> __device__ __forceinline__ void ring_advance(int* slot) {
    constexpr int M = Lat<Q>::M;
#pragma unroll
    for (int c = 0; c <= 2 * M; ++c) slot[c] = slot[c] + 1 == ring_len<Q>(c - M) ? 0 : slot[c] + 1;
}

// Group 0: the columns x = X0 - M + t of the level-(n+1) rows Y0 - M .. Y1 + M - 1.  A row's loads are
// one straight run of instructions with no branch between them and the collision of the row before
// (a wait at a join would cost the whole latency every row); columns of an x-side's layers (EDGE
// tiles) differ in their lane's address only, rows of a y-side's layers have loops of their own.
template <int Q, typename T, int NT, bool PX, bool PY, bool EDGE>
__device__ __forceinline__ void pair_producer(const T* A, const PairArgs<T>& g, int X0, int Y0, int Y1, int t,
                                              T omega, T* ring) {
    constexpr int M = Lat<Q>::M;
    int slot[2 * M + 1];
#pragma unroll
    for (int c = 0; c <= 2 * M; ++c) slot[c] = 0;
    int x = X0 - M + t;   // columns that no output needs are clamped
    x = PX ? min(x, g.nx - 1 + M) : min(max(x, 0), g.nx - 1);
    unsigned xs[2 * M + 1];
#pragma unroll
    for (int c = -M; c <= M; ++c) xs[c + M] = (unsigned)(PX ? wrapi(x - c, g.nx) : min(max(x - c, 0), g.nx - 1));
    const bool lane = EDGE && (x < g.x0 || x > g.x1);   // a layer column
    const T* lp = x < g.x0 ? g.lay[0].p + x : g.lay[1].p + x;
    const unsigned lpitch = (unsigned)(x < g.x0 ? g.lay[0].pitch : g.lay[1].pitch);
    auto load = [&](int r, T* d) {   // pull of a bulk row
        const int rw = PY ? wrapi(r, g.ny) : r;
        unsigned long long pitch = g.pitch;   // (opaque: 37 multiples of it kept across rows spill)
        asm("" : "+s"(pitch));
        const unsigned st = lane ? lpitch : (unsigned)pitch;   // EDGE: per lane a row address and a plane stride
        const T* lrow = lp + (long long)rw * Q * (long long)lpitch;
#pragma unroll
        for (int c = -M; c <= M; ++c) {
            const int ys = PY ? wrapi(rw - c, g.ny) : rw - c;
            const T* Ar = A + (unsigned long long)ys * Q * pitch;
            const T* Al = EDGE && lane ? lrow : Ar;
#pragma unroll
            for (int i = 0; i < Q; ++i) {
                if (cy<Q>(i) != c) continue;
                if (EDGE) d[i] = Al[(unsigned)i * st + (lane ? 0u : xs[cx<Q>(i) + M])];
                else d[i] = (Ar + (unsigned long long)i * pitch)[xs[cx<Q>(i) + M]];
            }
        }
    };
    auto hand_over = [&](const T* d) {
        each<Q>([&](auto I) { constexpr int i = I, o = ring_of<Q>(i), c = cy<Q>(i) + M; ring[(o + slot[c]) * NT + t] = d[i]; });
        lds_barrier();
        lds_barrier();
        ring_advance<Q>(slot);
    };
    // rows of a y-side's layers (all their columns, corner blocks included)
    auto lay_rows = [&](int r, int end, const View<T>& v) {
        for (; r < end; ++r) {
            const T* L = v.p + (long long)r * Q * (long long)v.pitch + xs[M];
            T d[Q];
#pragma unroll
            for (int i = 0; i < Q; ++i) d[i] = L[(unsigned long long)i * v.pitch];
            hand_over(d);
        }
    };
    const int rb = PY ? Y0 - M : max(Y0 - M, g.y0), re = PY ? Y1 + M : min(Y1 + M, g.y1 + 1);   // bulk rows
    // row r: d holds its pulled populations; those of row r + 1 are requested into n first, so that
    // they have the whole row's time to arrive (the last row requests itself again)
    auto row = [&](int r, T* d, T* n) {
        load(min(r + 1, re - 1), n);
        asm volatile("" ::: "memory");   // keep the requests here: not sunk to their use
        if (!lane) collide_dev<Q, T>(d, omega);
        hand_over(d);
    };
    if (!PY) lay_rows(Y0 - M, rb, g.lay[2]);
    T d0[Q], d1[Q];
    load(rb, d0);
    for (int r = rb; r < re; r += 2) {
        row(r, d0, d1);
        if (r + 1 < re) row(r + 1, d1, d0);
    }
    if (!PY) lay_rows(re, Y1 + M, g.lay[3]);
}

template <int Q, typename T, bool PX, bool PY>
__global__ __launch_bounds__((2 * pair_cols<Q, T>()), 1) void k_pair(const T* A, T* B, PairArgs<T> g) {
    constexpr int M = Lat<Q>::M, NT = pair_cols<Q, T>();
    __shared__ T ring[ring_slots<Q>() * NT];
    // work-group b runs on XCD b % 8: each XCD takes a contiguous range of tiles, x fastest, so that
    // the halo columns of neighbouring tiles meet in one L2
    const unsigned n8 = gridDim.x >> 3, rem = gridDim.x & 7u, k8 = blockIdx.x & 7u;
    const unsigned tile = k8 * n8 + min(k8, rem) + (blockIdx.x >> 3);
    const int seg = (int)(tile / (unsigned)g.ntx), tx = (int)(tile - (unsigned)seg * (unsigned)g.ntx);
    const int X0 = tx * g.wo;
    const int nr = g.y1 - g.y0 + 1;
    const int Y0 = g.y0 + (int)((long long)seg * nr / g.nseg), Y1 = g.y0 + (int)((long long)(seg + 1) * nr / g.nseg);
    const int group = __builtin_amdgcn_readfirstlane((int)threadIdx.x / NT);
    const int t = (int)threadIdx.x - group * NT;
    const T omega = sizeof(T) == 4 ? (T)g.omega_f : (T)g.omega_d;
    if (group == 0) {
        // the row hangs on this group's chain (loads, collision, hand-over): it issues first (the pass
        // alone 2 % faster on D2Q37 FP32, 4 % on D2Q17 FP32)
        __builtin_amdgcn_s_setprio(2);
        // tiles that hold layer columns take the loads with per-lane addresses
        if (!PX && (X0 - M < g.x0 || X0 - M + NT - 1 > g.x1)) pair_producer<Q, T, NT, PX, PY, true>(A, g, X0, Y0, Y1, t, omega, ring);
        else pair_producer<Q, T, NT, PX, PY, false>(A, g, X0, Y0, Y1, t, omega, ring);
    } else {
        const int x = X0 + t;
        const bool act = t < g.wo && x >= g.x0 && x <= g.x1;
        const int tc = min(t, NT - 1 - 2 * M) + M;   // its column among the NT
        int slot[2 * M + 1];
#pragma unroll
        for (int c = 0; c <= 2 * M; ++c) slot[c] = 0;
        for (int r = Y0 - M; r < Y1 + M; ++r) {
            const int y = r - M;
            ring_advance<Q>(slot);   // the oldest slots: the rows this output pulls from
            T e[Q];
            lds_barrier();
            if (y >= Y0) {
                each<Q>([&](auto I) {
                    constexpr int i = I, o = ring_of<Q>(i), c = cy<Q>(i) + M, dx = cx<Q>(i);
                    e[i] = ring[(o + slot[c]) * NT + tc - dx];
                });
            }
            lds_barrier();
            if (y >= Y0 && act) {
                collide_dev<Q, T>(e, omega);
                T* Bo = B + pix<Q>(g.pitch, 0, x, y);
#pragma unroll
                for (int i = 0; i < Q; ++i) __builtin_nontemporal_store(e[i], Bo + (unsigned long long)i * g.pitch);
            }
        }
    }
}

// ------------------------------------------------------------------ boundary launches of a pair
// One level of the sides, apart from the bulk.  TOC (n -> n + 1): the sides read A and write their
// layers into the band buffers; the work-groups from nbnd on compute the bulk nodes of the bands
// (x-bands: 16 rows of 16 lanes each, the bw - M columns next to the layers; y-bands: 256 nodes of
// one of the bw - M rows).  Otherwise (n + 1 -> n + 2): the sides read their band and write B.
template <typename T> struct BandArgs {
    View<T> src[4];      // per side: what its work-groups read
    int nbx, nby;        // TOC: work-groups per x-band, per y-band
    int xb[2], yb[2];    // TOC: which sides have a band
};

template <int Q, typename T, bool TOC, typename D>
__global__ __launch_bounds__(256, 2) void k_bnd(BandArgs<T> v, D dst, BndArgs a, BulkArgs g, int nbnd) {
    constexpr int M = Lat<Q>::M;
    int b = (int)blockIdx.x;
    if (b < nbnd) {
        boundary_job<Q, T, false>([&](int s) { return s == 0 ? v.src[0] : s == 1 ? v.src[1] : s == 2 ? v.src[2] : v.src[3]; }, dst, a, b);
        return;
    }
    if constexpr (TOC) {
        b -= nbnd;
        int x, y;
        const int nx2 = v.nbx * (v.xb[0] + v.xb[1]);
        if (b < nx2) {
            const bool hi = !v.xb[0] || b >= v.nbx;
            const int t = hi && v.xb[0] ? b - v.nbx : b, col = (int)(threadIdx.x & 15);
            if (col >= BW<Q> - M) return;
            x = hi ? g.x1 - col : g.x0 + col;
            y = g.y0 + t * 16 + (int)(threadIdx.x >> 4);
            if (y > g.y1) return;
        } else {
            b -= nx2;
            const bool hi = !v.yb[0] || b >= v.nby;
            const int t = hi && v.yb[0] ? b - v.nby : b;
            const int row = t % (BW<Q> - M);
            x = t / (BW<Q> - M) * 256 + (int)threadIdx.x;
            y = hi ? g.y1 - row : g.y0 + row;
            if (x < g.x0 || x > g.x1) return;
            if (!a.xper && (x < BW<Q> || x >= a.nx - BW<Q>)) return;   // in an x-band, which writes both
        }
        const View<T> A = v.src[0];
        T d[Q];
#pragma unroll
        for (int i = 0; i < Q; ++i) {
            int xs = x - cx<Q>(i), ys = y - cy<Q>(i);
            if (a.xper) xs = wrapi(xs, a.nx);
            if (a.yper) ys = wrapi(ys, a.ny);
            d[i] = A.p[pix<Q>(A.pitch, i, xs, ys)];
        }
        collide_dev<Q, T>(d, sizeof(T) == 4 ? (T)g.omega_f : (T)g.omega_d);
        dst.template put<Q>(x, y, [&](int i) { return d[i]; });
    }
}

}  // namespace lbm
