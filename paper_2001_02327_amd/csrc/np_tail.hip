// The coarse tail of a V-cycle (gfx950): the smallest multigrid levels, from a level
// Lt whose data and that of every coarser level fit in LDS together, down to the
// one-point level and back, in one workgroup: as separate launches their cost would
// be launch latency, not work.  Same operations in the same order and arithmetic as
// the per-level kernels: n_pre sweeps on Lt; per level down, the restriction
// (correction cleared) and n_pre sweeps; per level up, the prolongation and n_post
// sweeps.  Each level lives in LDS in natural order (x fastest) on its box of N_a + 2
// points per axis; the ghost slots are never written.
//
// What bounds it: the chain of some 35 dependent phases (a half sweep, a residual, a
// restriction, a prolongation), each an LDS round trip, seven additions and a
// barrier: 500 cycles per half sweep, 800 for a level's addresses, 1200 to 2700 for
// a transfer between levels.  So a thread owns a slot of the level (the two colours'
// points of the same place in a row), finds its neighbours' addresses and ghost
// factors once per visit of a level and keeps them in registers; the first red half
// sweep from zero, which reads no neighbour, is done where the right-hand side is
// formed; a restriction is one phase of residuals on every fine point and one of sums
// (a coarse point that formed its children's residuals one after the other took 6000
// cycles); and levels of at most 64 slots run in the first wavefront alone, without
// barriers.  Measured, V(2,1) in FP64 from 9^3 points: 20.4 -> 12.4 us; FP32 V(1,2) from 9^3:
// 11 us (17^3 in it, as before: 34.5 -> 35 us, four slots per thread).
#include <algorithm>
#include <type_traits>

#include "np_device.h"

// products with a ghost factor are rounded before they are added
#pragma clang fp contract(off)

namespace np {

namespace {

template <typename C>
struct TailLevel {
    int N[3];     // active points per axis
    int off;      // LDS element offset of u; f follows one box later
    int box;      // points of the box
    int cnt;      // slots: (N_x + 1) / 2 per row
    float rS, rN1;  // 1 / slots per row, 1 / N_y (index decoding)
    C h2, inv_h2;   // smoother factor (2^L h)^2 and its inverse
    GRule<C> gr;
};

template <typename C>
struct TailParams {
    TailLevel<C> lv[kTailMaxLevels];  // levels Lt .. Lt + nlev - 1 (the last has one point along some axis)
    int nlev;
    int nmulti;  // levels before the first of at most 64 slots
    int toff;    // LDS element offset of the residuals
    int n_pre, n_post;
};

// q = a / N and a % N for 0 <= a < 2^22 through a float reciprocal (rN = 1/N,
// loop-invariant) corrected by one step, instead of an integer division
__device__ __forceinline__ int divmod_small(int a, int N, float rN, int& rem)
{
    int q = (int)((float)a * rN);
    int r = a - q * N;
    if (r < 0) {
        q--;
        r += N;
    } else if (r >= N) {
        q++;
        r -= N;
    }
    rem = r;
    return q;
}

// A thread's point of a level: its element index and its neighbours' (below and above
// along each axis), a ghost neighbour by the point its value comes from and the factor.
template <int D, typename C>
struct TailPoint {
    int i, idx;
    bool on;
    int a[2 * D];
    C f[2 * D];
};

template <int D, typename C>
struct TailSlot {
    int j, k;
    TailPoint<D, C> p[2];  // by colour
};

template <int D, typename C>
__device__ __forceinline__ TailSlot<D, C> tail_slot(const TailLevel<C>& v, int t)
{
    TailSlot<D, C> s;
    const bool on = t < v.cnt;
    const int tt = on ? t : 0;
    const int hs = (v.N[0] + 1) >> 1;
    int sl;
    const int row = divmod_small(tt, hs, v.rS, sl);
    s.j = 1 + row;
    s.k = 0;
    if constexpr (D == 3) {
        int rj;
        s.k = 1 + divmod_small(row, v.N[1], v.rN1, rj);
        s.j = 1 + rj;
    }
    const int Qx = v.N[0] + 2, Qxy = Qx * (v.N[1] + 2);
    const int st[3] = {1, Qx, Qxy};
#pragma unroll
    for (int c = 0; c < 2; c++) {
        TailPoint<D, C>& p = s.p[c];
        p.i = 1 + ((1 + s.j + s.k + D + c) & 1) + 2 * sl;
        p.on = on && p.i <= v.N[0];
        p.idx = v.off + s.k * Qxy + s.j * Qx + p.i;
        const int q[3] = {p.i, s.j, s.k};
#pragma unroll
        for (int ax = 0; ax < D; ax++) {
            const bool lo = q[ax] == 1, hi = q[ax] == v.N[ax], x1 = v.gr.xn1[ax];
            const int al = lo ? p.idx : p.idx - st[ax];
            const C fl = lo ? (C)-1 : (C)1;
            p.a[2 * ax] = al;
            p.f[2 * ax] = fl;
            p.a[2 * ax + 1] = hi ? (x1 ? al : p.idx) : p.idx + st[ax];
            p.f[2 * ax + 1] = hi ? (x1 ? -fl : v.gr.coef[ax]) : (C)1;
        }
    }
    return s;
}

template <int D, typename C>
__device__ __forceinline__ C tail_sum(const C* lds, const TailPoint<D, C>& p)
{
    C n[2 * D];
#pragma unroll
    for (int e = 0; e < 2 * D; e++) n[e] = lds[p.a[e]];
    C s = p.f[0] * n[0] + p.f[1] * n[1];
#pragma unroll
    for (int e = 2; e < 2 * D; e++) s = s + p.f[e] * n[e];
    return s;
}

// Where the residuals of a coarse point's children lie (fine level of Nf points in
// natural order): the first child's and the steps to the second one along each axis, 0
// where that is outside the fine level (what is read instead is dropped).  The slot past an
// odd N_x (of the coarse level) holds no point: it takes the last point's children, so
// that every read stays inside the fine level's residuals.
struct TailKids {
    int at, dx, dy, dz;
    bool inx, iny, inz;
};

template <int D>
__host__ __device__ __forceinline__ TailKids tail_kids(int i, int j, int k, int N, const int (&Nf)[3])
{
    const int i0 = 2 * (i < N ? i : N) - 2, j0 = 2 * j - 2, k0 = D == 3 ? 2 * k - 2 : 0;
    TailKids q;
    q.inx = i0 + 1 < Nf[0];
    q.iny = j0 + 1 < Nf[1];
    q.inz = D == 3 && k0 + 1 < Nf[2];
    q.at = (k0 * Nf[1] + j0) * Nf[0] + i0;
    q.dx = q.inx ? 1 : 0;
    q.dy = q.iny ? Nf[0] : 0;
    q.dz = q.inz ? Nf[0] * Nf[1] : 0;
    return q;
}

// a level's parameters from LDS into scalar registers
template <typename C>
__device__ __forceinline__ TailLevel<C> tail_uniform(const TailLevel<C>& level)
{
    static_assert(sizeof(TailLevel<C>) % 4 == 0, "moved by words");
    union {
        TailLevel<C> v;
        int w[sizeof(TailLevel<C>) / 4];
    } x;
    x.v = level;
#pragma unroll
    for (unsigned i = 0; i < sizeof(TailLevel<C>) / 4; i++) x.w[i] = __builtin_amdgcn_readfirstlane(x.w[i]);
    return x.v;
}

// A visit of a level by the workgroup, or by its first wavefront alone (not MULTI);
// R slots per thread.
template <int D, int R, bool MULTI, typename C>
struct TailVisit {
    C* const lds;
    TailLevel<C> v;
    TailSlot<D, C> s[R];

    __device__ __forceinline__ void sync()
    {
        if constexpr (MULTI) lds_barrier();
        else __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");  // LDS serves a wavefront in order
    }

    // f(slot) of the thread's slots
    template <typename Fn>
    __device__ __forceinline__ void each(Fn f)
    {
#pragma unroll
        for (int r = 0; r < R; r++)
            if (r == 0 || r * (int)blockDim.x < v.cnt) f(s[r], r);
    }

    __device__ __forceinline__ void visit(const TailLevel<C>& level)
    {
        v = tail_uniform(level);
        each([&](TailSlot<D, C>& q, int r) { q = tail_slot<D, C>(v, (int)threadIdx.x + r * (int)blockDim.x); });
    }

    // sweeps; the first red half sweep is done already with `red_done`
    __device__ __forceinline__ void sweeps(int n, bool red_done)
    {
        const C inv2d = (C)(1.0 / (2.0 * D));
        const auto half = [&](int c) {
            each([&](const TailSlot<D, C>& q, int) {
                const TailPoint<D, C>& p = q.p[c];
                const C w = fma_t(-v.h2, lds[p.idx + v.box], tail_sum<D, C>(lds, p)) * inv2d;
                if (p.on) lds[p.idx] = w;
            });
            sync();
        };
#pragma unroll 1
        for (int it = 0; it < n; it++) {
            if (it > 0 || !red_done) half(0);
            half(1);
        }
    }

    // the residual of every point, in natural order at res
    __device__ __forceinline__ void residuals(C* res)
    {
        each([&](const TailSlot<D, C>& q, int) {
#pragma unroll
            for (int c = 0; c < 2; c++) {
                const TailPoint<D, C>& p = q.p[c];
                const C w = fma_t(-fma_t((C)(-2 * D), lds[p.idx], tail_sum<D, C>(lds, p)), v.inv_h2, lds[p.idx + v.box]);
                const int z = D == 3 ? q.k - 1 : 0;
                if (p.on) res[(z * v.N[1] + q.j - 1) * v.N[0] + p.i - 1] = w;
            }
        });
        sync();
    }

    // right-hand side f of a point, and where the level's first sweep starts
    __device__ __forceinline__ void start(const TailPoint<D, C>& p, int c, C f, int n_pre)
    {
        if (!p.on) return;
        lds[p.idx + v.box] = f;
        lds[p.idx] = c == 0 && n_pre > 0 ? ((C)0 - v.h2 * f) * (C)(1.0 / (2.0 * D)) : (C)0;
    }

    // right-hand side from the residuals of the finer level
    __device__ __forceinline__ void restrict_from(const C* res, const TailLevel<C>& fine, int n_pre)
    {
        const int Nf[3] = {__builtin_amdgcn_readfirstlane(fine.N[0]), __builtin_amdgcn_readfirstlane(fine.N[1]),
                           __builtin_amdgcn_readfirstlane(fine.N[2])};
        C sum[R][2];
        each([&](const TailSlot<D, C>& q, int r) {
#pragma unroll
            for (int c = 0; c < 2; c++) {
                const TailPoint<D, C>& p = q.p[c];
                const TailKids kid = tail_kids<D>(p.i, q.j, q.k, v.N[0], Nf);
                C ch[1 << D];
#pragma unroll
                for (int e = 0; e < (1 << D); e++)
                    ch[e] = res[kid.at + ((e & 1) ? kid.dx : 0) + ((e & 2) ? kid.dy : 0) + ((e & 4) ? kid.dz : 0)];
                C w = 0;
#pragma unroll
                for (int e = 0; e < (1 << D); e++) {
                    const bool in = (!(e & 1) || kid.inx) && (!(e & 2) || kid.iny) && (!(e & 4) || kid.inz);
                    w += in ? ch[e] : (C)0;
                }
                sum[r][c] = w * (C)(D == 3 ? 0.125 : 0.25);
            }
        });
        each([&](const TailSlot<D, C>& q, int r) {
#pragma unroll
            for (int c = 0; c < 2; c++) start(q.p[c], c, sum[r][c], n_pre);
        });
        sync();
    }

    // plus the interpolated correction of the next coarser level c
    __device__ __forceinline__ void prolong_from(const TailLevel<C>& coarse)
    {
        const TailLevel<C> cv = tail_uniform(coarse);
        const int Qx = cv.N[0] + 2, Qxy = Qx * (cv.N[1] + 2);
        const auto axis = [&](int q, int ax, AxisNb<C>& par, AxisNb<C>& nb) {
            par = axis_nb((q + 1) >> 1, cv.N[ax], cv.gr, ax);
            nb = axis_nb(((q + 1) >> 1) + ((q & 1) ? -1 : 1), cv.N[ax], cv.gr, ax);
            if (!par.ghost) par.fac = (C)1;
            if (!nb.ghost) nb.fac = (C)1;
        };
        each([&](const TailSlot<D, C>& q, int) {
            AxisNb<C> y[2], z[2];
            axis(q.j, 1, y[0], y[1]);
            if constexpr (D == 3) axis(q.k, 2, z[0], z[1]);
            C e[2][1 << D], u[2], fx[2][2];
#pragma unroll
            for (int c = 0; c < 2; c++) {
                const TailPoint<D, C>& p = q.p[c];
                AxisNb<C> x[2];
                axis(p.on ? p.i : 1, 0, x[0], x[1]);
#pragma unroll
                for (int m = 0; m < (1 << D); m++) {
                    int at = cv.off + y[(m >> 1) & 1].q * Qx + x[m & 1].q;
                    if constexpr (D == 3) at += z[m >> 2].q * Qxy;
                    e[c][m] = lds[at];
                }
                u[c] = lds[p.idx];
                fx[c][0] = x[0].fac;
                fx[c][1] = x[1].fac;
            }
#pragma unroll
            for (int c = 0; c < 2; c++) {
#pragma unroll
                for (int m = 0; m < (1 << D); m++) {
                    e[c][m] = y[(m >> 1) & 1].fac * (fx[c][m & 1] * e[c][m]);
                    if constexpr (D == 3) e[c][m] = z[m >> 2].fac * e[c][m];
                }
                const C(&g)[1 << D] = e[c];
                C w = prolong34(prolong34(g[0], g[1]), prolong34(g[2], g[3]));
                if constexpr (D == 3) w = prolong34(w, prolong34(prolong34(g[4], g[5]), prolong34(g[6], g[7])));
                if (q.p[c].on) lds[q.p[c].idx] = u[c] + w;
            }
        });
        sync();
    }
};

template <int D, int R, typename C>
__global__ void __launch_bounds__(kTailThreads) k_coarse_tail(TailParams<C> Pk, SGrid g0, const C* __restrict__ fg,
                                                              C* __restrict__ ug)
{
    extern __shared__ __align__(16) unsigned char tail_lds[];
    __shared__ TailParams<C> P;
    if (batch_idle(g0)) return;
    fg = batch_at(fg, g0);
    ug = batch_at(ug, g0);
    // The parameters move to LDS in one go: read level by level each visit of a new level
    // waited for them
    {
        using Word = const uint32_t __attribute__((address_space(4)))*;
        const Word k = (Word)__builtin_amdgcn_kernarg_segment_ptr();
        static_assert(sizeof(P) % 4 == 0, "copied by words");
        for (unsigned t = threadIdx.x; t < sizeof(P) / 4; t += blockDim.x) reinterpret_cast<uint32_t*>(&P)[t] = k[t];
        __syncthreads();
    }
    C* const lds = reinterpret_cast<C*>(tail_lds);
    C* const res = lds + __builtin_amdgcn_readfirstlane(P.toff);
    const int nm = __builtin_amdgcn_readfirstlane(P.nmulti), nlev = __builtin_amdgcn_readfirstlane(P.nlev);
    const int n_pre = __builtin_amdgcn_readfirstlane(P.n_pre), n_post = __builtin_amdgcn_readfirstlane(P.n_post);
    const int last = 2 * (nlev - 1);
    const auto body = [&](auto& m, int step) {
        const bool down = step < nlev;
        const int a = down ? step : last - step;
        m.visit(P.lv[a]);
        if (step == 0) {
            m.each([&](const TailSlot<D, C>& q, int) {
                C f[2];
#pragma unroll
                for (int c = 0; c < 2; c++) f[c] = fg[q.p[c].on ? pos<D, C>(g0, q.p[c].i, q.j, q.k) : (size_t)0];
#pragma unroll
                for (int c = 0; c < 2; c++) m.start(q.p[c], c, f[c], n_pre);
            });
            m.sync();
        } else if (down) {
            m.restrict_from(res, P.lv[a - 1], n_pre);
        } else {
            m.prolong_from(P.lv[a + 1]);
        }
        m.sweeps(down ? n_pre : n_post, down);
        if (down && a + 1 < nlev) m.residuals(res);
        if (step == last)
            m.each([&](const TailSlot<D, C>& q, int) {
#pragma unroll
                for (int c = 0; c < 2; c++)
                    if (q.p[c].on) ug[pos<D, C>(g0, q.p[c].i, q.j, q.k)] = lds[q.p[c].idx];
            });
    };
#pragma unroll 1
    for (int step = 0; step <= last; step++) {
        const int a = step < nlev ? step : last - step;
        if (step >= nlev && a + 1 == nm) lds_barrier();  // the first wavefront's levels are done
        if (a < nm) {
            TailVisit<D, R, true, C> m{lds};
            body(m, step);
        } else if (threadIdx.x < 64) {
            TailVisit<D, 1, false, C> m{lds};
            body(m, step);
        }
    }
}

}  // namespace

static size_t tail_box(int dim, const int* N)
{
    const size_t qx = (size_t)N[0] + 2, qy = (size_t)N[1] + 2, qz = (size_t)N[2] + 2;
    return dim == 3 ? qx * qy * qz : qx * qy;
}

size_t coarse_tail_lds_bytes(int dim, const int (*N)[3], int nlev, size_t esz)
{
    size_t e = 0;
    for (int a = 0; a < nlev; a++) e += 2 * tail_box(dim, N[a]);
    return e * esz;
}

int coarse_tail_slots(int dim, const int* N) { return (N[0] + 1) / 2 * N[1] * (dim == 3 ? N[2] : 1); }

template <typename T>
int launch_coarse_tail(int dim, hipStream_t st, int nlev, const int (*N)[3], const double* h, const Rule3* rule,
                       int n_pre, int n_post, SGrid g0, const T* f0, T* u0)
{
    if (nlev < 1 || nlev > kTailMaxLevels) return -1;
    if (coarse_tail_lds_bytes(dim, N, nlev, sizeof(T)) > kTailLdsBytes) return -1;
    TailParams<T> P{};
    P.nlev = nlev;
    P.n_pre = n_pre;
    P.n_post = n_post;
    int off = 0;
    for (int a = 0; a < nlev; a++) {
        TailLevel<T>& v = P.lv[a];
        for (int ax = 0; ax < 3; ax++) v.N[ax] = ax < dim ? N[a][ax] : 1;
        v.off = off;
        v.box = (int)tail_box(dim, N[a]);
        off += 2 * v.box;
        v.cnt = coarse_tail_slots(dim, N[a]);
        v.rS = 1.0f / (float)((v.N[0] + 1) / 2);
        v.rN1 = 1.0f / (float)v.N[1];
        v.h2 = (T)(h[a] * h[a]);
        v.inv_h2 = (T)(1.0 / (h[a] * h[a]));
        v.gr = grule<T>(rule[a]);
        if (v.cnt > 64) P.nmulti = a + 1;
    }
    P.toff = off;
    // the residuals: of the largest level at most
    const size_t bytes = (size_t)(off + N[0][0] * N[0][1] * (dim == 3 ? N[0][2] : 1)) * sizeof(T);
    const int nt = std::min(kTailThreads, ceil_div(P.lv[0].cnt, 64) * 64);
    const int slots = ceil_div(P.lv[0].cnt, nt);  // of a thread; the boxes' u and f fill 64 KB, so two at most in FP64, four in FP32
    const auto go = [&](auto d, auto r) {
        hipLaunchKernelGGL((k_coarse_tail<d.value, r.value, T>), dim3(1, g0.nb), dim3(nt), bytes, st, P, g0, f0, u0);
    };
    const auto by_slots = [&](auto d) {
        if (slots <= 1) go(d, std::integral_constant<int, 1>{});
        else if (slots <= 2) go(d, std::integral_constant<int, 2>{});
        else if constexpr (sizeof(T) == 4) go(d, std::integral_constant<int, 4>{});
    };
    if (slots > (sizeof(T) == 4 ? 4 : 2)) return -1;
    if (dim == 3) by_slots(std::integral_constant<int, 3>{});
    else by_slots(std::integral_constant<int, 2>{});
    return 0;
}

template int launch_coarse_tail<float>(int, hipStream_t, int, const int (*)[3], const double*, const Rule3*, int, int,
                                       SGrid, const float*, float*);
template int launch_coarse_tail<double>(int, hipStream_t, int, const int (*)[3], const double*, const Rule3*, int, int,
                                        SGrid, const double*, double*);

}  // namespace np
