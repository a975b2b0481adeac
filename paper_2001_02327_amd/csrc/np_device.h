// Device helpers shared by the kernels of the nested-grid multigrid solver
// (np_kernels.hip, np_tile.hip, np_tile2.hip, np_stream.hip, np_tail.hip): work numbering, lane shifts, colour-split
// indexing, maximum reductions, the ghost rule of the coarse levels.
#pragma once

#include "np_internal.h"

namespace np {

namespace {

constexpr int kBlock = 256;

__host__ __device__ inline int ceil_div(long a, long b) { return (int)((a + b - 1) / b); }

// Workgroups are dealt to the 8 XCDs of the chip round-robin (workgroup b runs
// on XCD b % 8).  Renumber them so that XCD x processes one contiguous run of
// logical blocks: stencil neighbours (rows above/below, planes in front/behind)
// are then fetched into the same XCD's L2 instead of eight different ones.
__device__ __forceinline__ long xcd_block()
{
    long nb = gridDim.x, b = blockIdx.x;
    long q = nb >> 3, r = nb & 7, x = b & 7, k = b >> 3;
    return x * q + (x < r ? x : r) + k;
}

// Two consecutive elements moved by one load or store of twice the width.
template <typename T>
struct alignas(2 * sizeof(T)) Pair {
    T a, b;
};

// Stores marked non-temporal, for FP64 data written once and not read again
// before much more than the caches hold has passed through them (the updated
// potential of the defect-correction pass, the forces, the coarse-to-fine
// fill): they then do not displace what the next kernels read.
__device__ __forceinline__ void store_nt(double* p, double v) { __builtin_nontemporal_store(v, p); }
__device__ __forceinline__ void store_nt(Pair<double>* p, const Pair<double>& v)
{
    typedef double d2_t __attribute__((ext_vector_type(2)));
    const d2_t x = {v.a, v.b};
    __builtin_nontemporal_store(x, (d2_t*)p);
}
constexpr bool kFillNt = true;  // non-temporal stores in the level setup kernels as well
// load of FP64 data read once and not again soon (the right-hand side in the
// defect-correction pass)
__device__ __forceinline__ Pair<double> load_nt(const Pair<double>* p)
{
    typedef double d2_t __attribute__((ext_vector_type(2)));
    const d2_t x = __builtin_nontemporal_load((const d2_t*)p);
    return Pair<double>{x.x, x.y};
}
constexpr bool kDcLoadNt = true;

// Consecutive level-0 kernels of a V-cycle run their z-chunks in alternating
// directions (rev: the logical block order reversed), so that each starts on
// the planes the previous one touched last, which the memory-side cache still
// holds.  The direction changes the order of the work only, never its result.
constexpr bool kAlternateZ = true;

__device__ __forceinline__ int zmarch_block(int rev)
{
    const int lb = (int)xcd_block();
    return (kAlternateZ && rev) ? (int)gridDim.x - 1 - lb : lb;
}

// Value of the previous (lane - 1) and next (lane + 1) lane of the wave by a
// DPP wave shift; lane 0 (previous) and lane 63 (next) get 0.
__device__ __forceinline__ unsigned dpp_prev(unsigned v)
{
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xf, 0xf, true);  // wave_shr:1
}
__device__ __forceinline__ unsigned dpp_next(unsigned v)
{
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x130, 0xf, 0xf, true);  // wave_shl:1
}
__device__ __forceinline__ float dpp_prev(float x) { return __uint_as_float(dpp_prev(__float_as_uint(x))); }
__device__ __forceinline__ float dpp_next(float x) { return __uint_as_float(dpp_next(__float_as_uint(x))); }
__device__ __forceinline__ double dpp_prev(double x)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
    const unsigned long long lo = dpp_prev((unsigned)b), hi = dpp_prev((unsigned)(b >> 32));
    return __builtin_bit_cast(double, lo | (hi << 32));
}
__device__ __forceinline__ double dpp_next(double x)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
    const unsigned long long lo = dpp_next((unsigned)b), hi = dpp_next((unsigned)(b >> 32));
    return __builtin_bit_cast(double, lo | (hi << 32));
}

// Strip ordering of a 3-D box of points (x fastest): the y range is cut into
// strips of R rows and logical blocks run over (strip, z, block of the strip
// plane).  With the XCD-contiguous numbering above, every XCD walks whole
// strips plane by plane, so the planes a stencil revisits (z-neighbours) and
// the rows it shares (y-neighbours) are still in that XCD's L2.
struct Strip {
    int nxa, nya, nza;  // box extents
    int R;              // rows per strip
    int B;              // blocks per strip plane
};

inline Strip make_strip(int nxa, int nya, int nza, int nstrip)
{
    Strip s;
    s.nxa = nxa;
    s.nya = nya;
    s.nza = nza;
    s.R = (nya + nstrip - 1) / nstrip;
    s.B = (int)(((long)s.R * nxa + kBlock - 1) / kBlock);
    return s;
}

__device__ __forceinline__ bool strip_point(const Strip& s, int& x, int& y, int& z)
{
    const int lb = (int)xcd_block();
    const int per = s.nza * s.B;
    const int st = lb / per;
    const int rem = lb - st * per;
    z = rem / s.B;
    const int blk = rem - z * s.B;
    const int tin = blk * kBlock + threadIdx.x;
    const int rr = tin / s.nxa;
    x = tin - rr * s.nxa;
    y = st * s.R + rr;
    return rr < s.R && y < s.nya;
}

// Patch batches (SGrid::nb): a multigrid launch over nb patches of one grid
// runs patch blockIdx.y; its arrays start blockIdx.y * bs elements in, and a
// patch whose flag in act is 0 has stopped iterating: its blocks return at
// once (a block-uniform exit, before any barrier).
__device__ __forceinline__ bool batch_idle(const SGrid& g) { return g.act && !g.act[blockIdx.y]; }

template <typename T>
__device__ __forceinline__ T* batch_at(T* p, const SGrid& g)
{
    return p ? p + (size_t)blockIdx.y * g.bs : p;
}

template <int D>
__device__ __forceinline__ int colour_of(int pi, int pj, int pk)
{
    return (pi + pj + pk + D) & 1;
}

__device__ __forceinline__ size_t row_base(const SGrid& g, int pj, int pk)
{
    return (size_t)pk * g.ps + (size_t)pj * g.hx;
}

template <int D, typename T>
__device__ __forceinline__ T at(const T* __restrict__ a, const SGrid& g, int pi, int pj, int pk)
{
    return a[(size_t)colour_of<D>(pi, pj, pk) * g.cs + row_base(g, pj, pk) + (pi >> 1)];
}

template <int D, typename T>
__device__ __forceinline__ size_t pos(const SGrid& g, int pi, int pj, int pk)
{
    return (size_t)colour_of<D>(pi, pj, pk) * g.cs + row_base(g, pj, pk) + (pi >> 1);
}

// Maximum of non-negative doubles through their bit patterns: the unsigned
// order of the patterns is the numeric order, +inf above every finite value
// and a (positive) NaN above +inf, so NaN and Inf survive the reduction.
__device__ __forceinline__ unsigned long long wave_max_u64(unsigned long long v)
{
    for (int off = 32; off > 0; off >>= 1) {
        unsigned long long o = __shfl_xor(v, off, 64);
        v = o > v ? o : v;
    }
    return v;
}

// Maximum of v over a block of NW wavefronts into *out.  Atomics on one address
// are served one after another, ~12 ns each: the 4096 blocks of a 1024^2 force
// test spent ~45 of its 52 us there.  So a block first reads *out (~6 ns each,
// 27 us for that test) and issues its atomic only when it would raise the
// maximum, which never falls during a kernel (a stale read costs a superfluous
// atomic at most); and the kernels that have little work per block run at most
// kReduceBlocks blocks in grid-stride loops (19 us for that test).  CHECK is off
// in the z-march passes, whose blocks end far enough apart (residual norm of a
// 258^3 level: 33.8 us without the read, 36.9 with it).
constexpr int kReduceBlocks = 512;
template <int NW, bool CHECK = true>
__device__ __forceinline__ void block_max_to_w(unsigned long long v, unsigned long long* out)
{
    __shared__ unsigned long long red[NW];
    v = wave_max_u64(v);
    int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) red[wave] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long m = red[0];
        for (int w = 1; w < NW; w++) m = red[w] > m ? red[w] : m;
        if (!CHECK || m > __hip_atomic_load(out, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(out, m);
    }
}

template <bool CHECK = true>
__device__ __forceinline__ void block_max_to(unsigned long long v, unsigned long long* out)
{
    block_max_to_w<kBlock / 64, CHECK>(v, out);
}

__device__ __forceinline__ unsigned long long abs_bits(double a)
{
    return (unsigned long long)__double_as_longlong(fabs(a));
}

// Residual f - (s - 2d u) / h^2 at a point (s: the sum of its 2d neighbours)
// with the rounding every residual-norm pass uses: one fused multiply-add
// forms s - 2d u, a second f - (s - 2d u) inv_h2.
__device__ __forceinline__ double resid(double f, double s, double u, double two_d, double inv_h2)
{
    return __fma_rn(-inv_h2, __fma_rn(-two_d, u, s), f);
}

template <typename T>
struct Compute { using type = T; };
template <>
struct Compute<__half> { using type = float; };

// Ghost rule of a multigrid level L >= 1 (Sec. 2.4): the layer outside the
// active points 1..N is anti-symmetric, e_0 = -e_1 on the left and on the right
// e_{N+1} = -e_{N-1} when x_N = 1, else coef * e_N; points outside along several
// axes compose the rule of each axis in the order x, y, z.  The kernels never
// store this layer: they evaluate it where they read it.  That gives the values
// a refresh before every half sweep would: a face ghost next to an active
// point p depends only on p itself or on the point beyond p on the same axis,
// which has the other colour, and neither changes before p's own update.
template <typename C>
struct GRule {
    int xn1[3];  // per axis: the last active centre sits at x_MG = 1
    C coef[3];   // per axis: the right-ghost coefficient otherwise
};

template <typename C>
GRule<C> grule(const Rule3& r)
{
    return GRule<C>{{r.xn1[0], r.xn1[1], r.xn1[2]}, {(C)r.coef[0], (C)r.coef[1], (C)r.coef[2]}};
}

// Value at padded point p of a level with a rule ghost layer (any point, ghost
// along any number of axes).  Factors are applied per axis in x, y, z order.
template <int D, typename T, typename C>
__device__ __forceinline__ C rule_at(const T* __restrict__ a, const SGrid& g, int pi, int pj, int pk,
                                     const GRule<C>& gr)
{
    const int Na[3] = {g.nx - 2, g.ny - 2, g.nz - 2};
    int p[3] = {pi, pj, pk};
    C fac[3] = {(C)1, (C)1, (C)1};
    bool sc[3] = {false, false, false};
    for (int ax = 0; ax < D; ax++) {
        const int N = Na[ax];
        if (p[ax] == 0) {
            p[ax] = 1;
            fac[ax] = (C)-1;
            sc[ax] = true;
        } else if (p[ax] == N + 1) {
            p[ax] = gr.xn1[ax] ? N - 1 : N;
            fac[ax] = gr.xn1[ax] ? (C)-1 : gr.coef[ax];
            sc[ax] = true;
        }
    }
    C v = (C)at<D>(a, g, p[0], p[1], p[2]);
    for (int ax = 0; ax < D; ax++)
        if (sc[ax]) v = fac[ax] * v;
    return v;
}

// Face-ghost substitution for a 7-point stencil at active index q (1..N) along
// axis ax: the neighbour below (q = 1) is -self; the neighbour above (q = N)
// is -(the neighbour below) when x_N = 1, else coef * self.
template <typename C>
__device__ __forceinline__ void rule_pair(int q, int N, C self, C& lo, C& hi, const GRule<C>& gr, int ax)
{
    if (q == 1) lo = -self;
    if (q == N) hi = gr.xn1[ax] ? -lo : gr.coef[ax] * self;
}

// Barrier that orders LDS only: __syncthreads also waits for every global load in
// flight.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// fused multiply-add in the type of its operands
__device__ __forceinline__ double fma_t(double a, double b, double c) { return __fma_rn(a, b, c); }
__device__ __forceinline__ float fma_t(float a, float b, float c) { return __fmaf_rn(a, b, c); }

// 3/4 of the parent plus 1/4 of the neighbour, with the rounding every
// prolongation kernel uses: one (a quarter of a value is exact)
template <typename C>
__device__ __forceinline__ C prolong34(C parent, C nb)
{
    return fma_t((C)0.75, parent, (C)0.25 * nb);
}

// Parent or neighbour of a fine point on one axis of a coarse level: its index
// after the rule, and the rule's factor where it is a ghost.
template <typename C>
struct AxisNb {
    int q;       // neighbour index after the rule
    C fac;       // rule factor
    bool ghost;  // the factor applies
};

template <typename C>
__device__ __forceinline__ AxisNb<C> axis_nb(int q, int N, const GRule<C>& gr, int ax)
{
    AxisNb<C> a{q, (C)1, false};
    if (q == 0) {
        a.q = 1;
        a.fac = (C)-1;
        a.ghost = true;
    } else if (q == N + 1) {
        a.q = gr.xn1[ax] ? N - 1 : N;
        a.fac = gr.xn1[ax] ? (C)-1 : gr.coef[ax];
        a.ghost = true;
    }
    return a;
}

template <typename C>
__device__ __forceinline__ AxisNb<C> axis_nb_clamped(int q, int N, const GRule<C>& gr, int ax)
{
    // q = N + 2 only beside a ghost parent, on the side it has no child: any
    // in-bounds value serves
    return axis_nb(q > N + 1 ? N + 1 : q, N, gr, ax);
}

}  // namespace

}  // namespace np
