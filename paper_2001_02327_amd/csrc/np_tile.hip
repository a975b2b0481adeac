// Fused V-cycle legs of a small 3-D multigrid level (gfx950).
//
// Kernels that each make one pass over a level (a half sweep, the residual and
// restriction, the prolongation) are bound by launch latency on the small levels:
// 4-5 us each, however little they do, eight or nine of them per level and
// cycle.  Here a whole leg of the cycle is one launch:
//   down: the pre-smoothing sweeps, the residual and its restriction;
//   up:   the prolongation and correction, the post-smoothing sweeps and (for
//         the stop test) the residual's max norm.
// A workgroup owns a block of 4 x 4 x 4 to 16 x 16 x 8 points and takes it through every half
// sweep of the leg in LDS, together with a halo one point wide per half sweep that
// follows (H in all), which it recomputes: a point at distance d from the block is
// relaxed only by the half sweeps whose values can still reach the block.  Halo
// values are read from arrays that no workgroup of the launch writes, so the result
// does not depend on the order of the workgroups.  Every operation and its order are
// those of the per-pass kernels (np_kernels.hip), so the iterates are the same bit
// for bit.
//
// Threads: a thread owns one compact column (h, y) of the region for both
// colours and a range of PZ planes; it keeps their right-hand sides and values in
// registers, and the potential of the region lies in LDS too for the neighbours in x and
// y and at the ends of the range (colour-split, so that lanes read consecutive elements):
// three loads per point.  A leg is bound by its half sweeps' LDS loads and additions
// (up to 1 us each): 8.6 us down and 5.5 us up for V(2,1) on 33^3 points in FP64, against
// 31 us in per-pass kernels.  In blocks of 8 x 8 x 8 points, with the columns' values read back from LDS (4.5 loads per
// point, 5.5 beside the boundary) and the boundary rule formed by selects per neighbour:
// 9.8 + 7.2 us against 9.1 + 6.6 (a half sweep 2300 cycles, 3000 beside the boundary); 65^3
// in wide blocks 15.3 + 9.6 against 13.4 + 8.6, FP32 V(1,2) up 13.0 against 11.9.
#include <type_traits>

#include "np_device.h"

// multiply-adds are written out, as in the other form of the legs
#pragma clang fp contract(off)

namespace np {

namespace {

// Region of a block of TX x TX x TZ points with a halo of H points: HC compact
// columns per row, RY rows, RZ planes; G ranges of PZ planes, WPG wavefronts each.
// The LDS holds a plane more on either side of the ranges, so that no z-neighbour
// needs a clamp (what is read there feeds no stored value).
template <int H_, int TX_, int TZ_, int G_, int PZ_>
struct TlShape {
    static constexpr int H = H_, TX = TX_, TZ = TZ_, G = G_, PZ = PZ_;
    static constexpr int HC = TX / 2 + (H | 1);  // the region starts at an odd x for even H
    static constexpr int RY = TX + 2 * H;
    static constexpr int RZ = TZ + 2 * H;
    static constexpr int NCOL = HC * RY;
    static constexpr int WPG = (NCOL + 63) / 64;
    static constexpr int NT = 64 * WPG * G;
    static constexpr int FRONT = NCOL + HC + 1;               // elements before the first plane
    static constexpr int CS = G * PZ * NCOL + 2 * FRONT;      // LDS elements per colour
    // planes whose loads are issued together
    static constexpr int SB = PZ <= 6 ? PZ : (PZ % 2 == 0 ? PZ / 2 : PZ);
    static_assert(G * PZ >= RZ && NT <= 1024 && PZ % SB == 0, "every plane has a thread");
};

// What a thread knows of its place in the region and of the level.
template <typename S>
struct TlPlace {
    int col, hg, pj, zl0, pk0;  // compact column, its global slot and row, first plane (in the region, global)
    bool in_col;
    int X0, Y0, Z0;             // first point of the block
    int Nx, Ny, Nz;

    __device__ __forceinline__ TlPlace(const SGrid& g, int nbx, int nby, int rev)
    {
        int lb = (int)xcd_block();
        if (rev) lb = (int)gridDim.x - 1 - lb;
        const int bx = lb % nbx, t = lb / nbx, by = t % nby, bz = t / nby;
        X0 = 1 + S::TX * bx;
        Y0 = 1 + S::TX * by;
        Z0 = 1 + S::TZ * bz;
        Nx = g.nx - 2;
        Ny = g.ny - 2;
        Nz = g.nz - 2;
        const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
        const int zg = wave / S::WPG;
        const int c = (wave - zg * S::WPG) * 64 + (int)(threadIdx.x & 63);
        in_col = c < S::NCOL;
        col = in_col ? c : S::NCOL - 1;
        const int ly = col / S::HC;
        hg = ((X0 - S::H) >> 1) + (col - ly * S::HC);
        pj = Y0 - S::H + ly;
        zl0 = zg * S::PZ;
        pk0 = Z0 - S::H + zl0;
    }
    // whether the block's region reaches the level's boundary
    __device__ __forceinline__ bool edge() const
    {
        return X0 - S::H < 2 || Y0 - S::H < 2 || Z0 - S::H < 2 || X0 + S::TX - 1 + S::H >= Nx ||
               Y0 + S::TX - 1 + S::H >= Ny || Z0 + S::TZ - 1 + S::H >= Nz;
    }
};

// A thread's masks for the points within rho of the block: its column's even
// and odd point, and the planes.
struct TlRange {
    bool v0, v1;
    int zlo, zhi;
};

template <typename S, typename P>
__device__ __forceinline__ TlRange tl_range(const P& p, int rho)
{
    TlRange r;
    const int x0 = 2 * p.hg, x1 = x0 + 1;
    const int xlo = max(1, p.X0 - rho), xhi = min(p.Nx, p.X0 + S::TX - 1 + rho);
    const bool y = p.in_col && p.pj >= max(1, p.Y0 - rho) && p.pj <= min(p.Ny, p.Y0 + S::TX - 1 + rho);
    r.v0 = y && x0 >= xlo && x0 <= xhi;
    r.v1 = y && x1 >= xlo && x1 <= xhi;
    r.zlo = max(1, p.Z0 - rho);
    r.zhi = min(p.Nz, p.Z0 + S::TZ - 1 + rho);
    return r;
}

// How a pass reads the x and y neighbours outside a thread's column in a block at the
// boundary: offsets from the point in the other colour's array and factors.  A ghost
// value is a factor times the point itself or the neighbour opposite, so a thread
// whose neighbour is a ghost reads that value's address instead; no test per point.
template <typename C>
struct TlNb {
    int xa, xb, y0, y1;      // x: in the thread's even and odd planes
    C fxa, fxb, fy0, fy1;
    bool ga, gb, far;        // the column's own x neighbour is a ghost, and (far) of the neighbour opposite
    C fg;
};

template <int COLOUR, typename S, typename C, typename P>
__device__ __forceinline__ TlNb<C> tl_nb(const P& p, int par0, const GRule<C>& gr)
{
    constexpr int self = COLOUR ? S::CS : -S::CS;  // from the other colour's array to this one's
    const C fx = gr.xn1[0] ? (C)-1 : gr.coef[0], fy = gr.xn1[1] ? (C)-1 : gr.coef[1];
    const bool lo = p.hg == 0, hi = 2 * p.hg == p.Nx, hi_odd = 2 * p.hg + 1 == p.Nx;
    TlNb<C> n;
    const int x1 = hi_odd ? (gr.xn1[0] ? 0 : self) : 1;  // the odd point's
    const C f1 = hi_odd ? fx : (C)1;
    n.xa = par0 ? x1 : -1;
    n.xb = par0 ? -1 : x1;
    n.fxa = par0 ? f1 : (C)1;
    n.fxb = par0 ? (C)1 : f1;
    n.ga = par0 ? lo : hi;
    n.gb = par0 ? hi : lo;
    n.far = hi && gr.xn1[0];
    n.fg = lo ? (C)-1 : fx;
    n.y0 = p.pj == 1 ? self : -S::HC;
    n.fy0 = p.pj == 1 ? (C)-1 : (C)1;
    n.y1 = p.pj == p.Ny ? (gr.xn1[1] ? -S::HC : self) : S::HC;
    n.fy1 = p.pj == p.Ny ? fy : (C)1;
    return n;
}

// One half sweep of COLOUR over the points within rho of the block, or (RESID)
// f - lap u at the block's points of that colour into rr.  uo, uw: the thread's column of
// the other colour and of this one, as they are in LDS; fv: its right-hand sides of this
// colour.  STORE: other threads read the result.  Every load of SB planes is issued before the first
// is used and nothing branches in between (points out of range are formed
// and dropped: their store goes to a slot in front of the array): with a branch
// per point the compiler put each point's loads behind it and every plane
// cost an LDS round trip and the chain of its additions, 14 us per leg on one block.
template <int COLOUR, bool RULE, bool EDGE, bool RESID, bool STORE, typename S, typename C, typename P>
__device__ __forceinline__ void tl_pass(C* R, C* B, const C (&uo)[S::PZ], C (&uw)[S::PZ], const C (&fv)[S::PZ], const P& p,
                                        int rho, C h2, C inv2d, const GRule<C>& gr, C (&rr)[S::PZ])
{
    const C* o = COLOUR ? R : B;
    C* w = COLOUR ? B : R;
    const TlRange r = tl_range<S>(p, rho);
    // parity term of the colour's point in the thread's first plane: x = 2 h + par
    const int par0 = (COLOUR + p.pj + p.pk0 + 3) & 1;
    const int dx0 = par0 ? 1 : -1;
    const bool va = par0 ? r.v1 : r.v0, vb = par0 ? r.v0 : r.v1;
    TlNb<C> nb;
    if constexpr (RULE && EDGE) nb = tl_nb<COLOUR, S>(p, par0, gr);
    if constexpr (RESID) {
#pragma unroll
        for (int j = 0; j < S::PZ; j++) rr[j] = (C)0;
    }
#pragma unroll
    for (int jb = 0; jb < S::PZ; jb += S::SB) {
        if (p.pk0 + jb > r.zhi || p.pk0 + jb + S::SB - 1 < r.zlo) continue;  // uniform over the wavefront
        const int at0 = (p.zl0 + jb) * S::NCOL + p.col;
        C ov[S::SB + 2], xo[S::SB], ya[S::SB], yb[S::SB];
#pragma unroll
        for (int j = 0; j < S::SB + 2; j++) {
            const int k = jb + j - 1;
            ov[j] = k >= 0 && k < S::PZ ? uo[k < 0 || k >= S::PZ ? 0 : k] : o[at0 + (j - 1) * S::NCOL];
        }
#pragma unroll
        for (int j = 0; j < S::SB; j++) {
            const int at = at0 + j * S::NCOL;
            if constexpr (RULE && EDGE) {
                xo[j] = o[at + (((jb + j) & 1) ? nb.xb : nb.xa)];
                ya[j] = o[at + nb.y0];
                yb[j] = o[at + nb.y1];
            } else {
                xo[j] = o[at + (((jb + j) & 1) ? -dx0 : dx0)];
                ya[j] = o[at - S::HC];
                yb[j] = o[at + S::HC];
            }
        }
        C v[S::SB];
#pragma unroll
        for (int j = 0; j < S::SB; j++) {
            C y0 = ya[j], y1 = yb[j], z0 = ov[j], z1 = ov[j + 2], xm = ov[j + 1], xp = xo[j];
            const C me = uw[jb + j];
            if constexpr (RULE && EDGE) {
                const bool odd = (jb + j) & 1;
                const C ghost = nb.fg * (nb.far ? xp : me);
                xp = (odd ? nb.fxb : nb.fxa) * xp;
                xm = (odd ? nb.gb : nb.ga) ? ghost : xm;
                y0 = nb.fy0 * y0;
                y1 = nb.fy1 * y1;
                rule_pair(p.pk0 + jb + j, p.Nz, me, z0, z1, gr, 2);
            }
            C s = xm + xp;
            s = s + y0;
            s = s + y1;
            s = s + z0;
            s = s + z1;
            if constexpr (RESID) v[j] = fma_t(-h2, fma_t((C)-6, me, s), fv[jb + j]);  // (h2: 1 / h^2)
            else v[j] = (fma_t(-h2, fv[jb + j], s) * inv2d);
        }
#pragma unroll
        for (int j = 0; j < S::SB; j++) {
            const int pk = p.pk0 + jb + j;
            const bool live = (((jb + j) & 1) ? vb : va) && pk >= r.zlo && pk <= r.zhi;
            if constexpr (RESID) {
                rr[jb + j] = live ? v[j] : (C)0;
            } else {
                uw[jb + j] = live ? v[j] : uw[jb + j];
                if constexpr (STORE) w[live ? at0 + j * S::NCOL : -S::FRONT] = v[j];
            }
        }
    }
}

template <int COLOUR, bool RULE, bool EDGE, bool STORE, typename S, typename C, typename P>
__device__ __forceinline__ void tl_sweep(C* R, C* B, C (&ur)[S::PZ], C (&ub)[S::PZ], const C (&fv)[S::PZ], const P& p,
                                         int rho, C h2, C inv2d, const GRule<C>& gr)
{
    C none[S::PZ];
    if constexpr (COLOUR) tl_pass<1, RULE, EDGE, false, STORE, S>(R, B, ur, ub, fv, p, rho, h2, inv2d, gr, none);
    else tl_pass<0, RULE, EDGE, false, STORE, S>(R, B, ub, ur, fv, p, rho, h2, inv2d, gr, none);
}

template <int COLOUR, bool RULE, bool EDGE, typename S, typename C, typename P>
__device__ __forceinline__ void tl_resid(C* R, C* B, C (&ur)[S::PZ], C (&ub)[S::PZ], const C (&fv)[S::PZ], const P& p,
                                         C inv_h2, const GRule<C>& gr, C (&rr)[S::PZ])
{
    if constexpr (COLOUR) tl_pass<1, RULE, EDGE, true, false, S>(R, B, ur, ub, fv, p, 0, inv_h2, (C)0, gr, rr);
    else tl_pass<0, RULE, EDGE, true, false, S>(R, B, ub, ur, fv, p, 0, inv_h2, (C)0, gr, rr);
}

// loads the thread's columns of both colours of a global array (0 outside the grid)
template <typename S, typename T, typename C, typename P>
__device__ __forceinline__ void tl_load(const T* __restrict__ a, const SGrid& g, const P& p, C (&r)[S::PZ], C (&b)[S::PZ])
{
    const bool ok = p.in_col && p.hg >= 0 && p.hg < g.hx && p.pj >= 0 && p.pj < g.ny;
    const size_t base = (size_t)p.pj * g.hx + p.hg;
#pragma unroll
    for (int j = 0; j < S::PZ; j++) {
        const int pk = p.pk0 + j;
        r[j] = (C)0;
        b[j] = (C)0;
        if (p.zl0 + j < S::RZ && pk >= 0 && pk < g.nz && ok) {
            r[j] = (C)a[(size_t)pk * g.ps + base];
            b[j] = (C)a[g.cs + (size_t)pk * g.ps + base];
        }
    }
}

// puts the thread's columns of both colours in LDS
template <typename S, typename C, typename P>
__device__ __forceinline__ void tl_keep(C* R, C* B, const P& p, const C (&r)[S::PZ], const C (&b)[S::PZ])
{
#pragma unroll
    for (int j = 0; j < S::PZ; j++)
        if (p.zl0 + j < S::RZ && p.in_col) {
            const int at = (p.zl0 + j) * S::NCOL + p.col;
            R[at] = r[j];
            B[at] = b[j];
        }
}

// The down leg.  WARM: from u_in (whose ghost layer is fixed, in memory);
// otherwise from zero, with the ghost layer zero or (RULE) given by the rule.  Writes
// the black points of the block to u_out (with RULE the red ones too, which the
// up leg's ghost values need) and the restricted residual to fc.
template <typename T, int NPRE, bool RULE, typename S>
__global__ void __launch_bounds__(S::NT)
k_tile_down3(const T* __restrict__ u_in, const T* __restrict__ f, SGrid g, T* __restrict__ u_out,
              T h2, T inv2d, T inv_h2,
              T scale, GRule<T> gr, SGrid gc, T* __restrict__ fc, int nbx,
              int nby, int rev)
{
    using C = T;
    constexpr bool WARM = !RULE;
    constexpr int H = S::H, TX = S::TX, TZ = S::TZ;
    static_assert(H == 2 * NPRE + WARM, "a halo point per half sweep that follows");
    static_assert(TX * TX * TZ <= 2 * S::CS, "the residuals fit in the region's LDS");
    __shared__ __align__(16) C lds[2 * S::CS];
    if (batch_idle(g)) return;
    u_in = batch_at(u_in, g);
    f = batch_at(f, g);
    u_out = batch_at(u_out, g);
    fc = batch_at(fc, gc);
    C* const R = lds + S::FRONT;
    C* const B = lds + S::CS + S::FRONT;
    const TlPlace<S> p(g, nbx, nby, rev);
    C fr[S::PZ], fb[S::PZ];
    tl_load<S>(f, g, p, fr, fb);
    C ur[S::PZ], ub[S::PZ];
    if constexpr (WARM) {
        const bool ok = p.in_col && p.hg >= 0 && p.hg < g.hx && p.pj >= 0 && p.pj < g.ny;
        const size_t base = (size_t)p.pj * g.hx + p.hg;
        const int x0 = 2 * p.hg;
        // red points are relaxed before they are read, except those of the ghost layer
        const bool row_ring = p.pj == 0 || p.pj == g.ny - 1;
        const int par0 = (p.pj + p.pk0 + 3) & 1;
#pragma unroll
        for (int j = 0; j < S::PZ; j++) {
            const int pk = p.pk0 + j;
            ur[j] = (C)0;
            ub[j] = (C)0;
            if (p.zl0 + j < S::RZ && pk >= 0 && pk < g.nz && ok) {
                ub[j] = (C)u_in[g.cs + (size_t)pk * g.ps + base];
                const int x = x0 + ((j & 1) ? par0 ^ 1 : par0);
                if (row_ring || pk == 0 || pk == g.nz - 1 || x == 0 || x == g.nx - 1)
                    ur[j] = (C)u_in[(size_t)pk * g.ps + base];
            }
        }
    } else {
        // the first red half sweep from zero needs the right-hand side only
        const TlRange r = tl_range<S>(p, H);
        const int par0 = (p.pj + p.pk0 + 3) & 1;
        const bool va = par0 ? r.v1 : r.v0, vb = par0 ? r.v0 : r.v1;
#pragma unroll
        for (int j = 0; j < S::PZ; j++) {
            const int pk = p.pk0 + j;
            const bool live = pk >= r.zlo && pk <= r.zhi && ((j & 1) ? vb : va);
            ur[j] = live ? (((C)0 - h2 * fr[j]) * inv2d) : (C)0;
            ub[j] = (C)0;
        }
    }
    tl_keep<S>(R, B, p, ur, ub);
    __syncthreads();
    C rr[S::PZ], rb[S::PZ];
    const auto leg = [&](auto edge) {
        constexpr bool E = decltype(edge)::value;
#pragma unroll
        for (int it = 0; it < NPRE; it++) {
            if (WARM || it > 0) {
                tl_sweep<0, RULE, E, true, S>(R, B, ur, ub, fr, p, 2 * (NPRE - it), h2, inv2d, gr);
                __syncthreads();
            }
            tl_sweep<1, RULE, E, true, S>(R, B, ur, ub, fb, p, 2 * (NPRE - it) - 1, h2, inv2d, gr);
            __syncthreads();
        }
        tl_resid<0, RULE, E, S>(R, B, ur, ub, fr, p, inv_h2, gr, rr);
        tl_resid<1, RULE, E, S>(R, B, ur, ub, fb, p, inv_h2, gr, rb);
    };
    if (RULE && p.edge()) leg(std::true_type{});
    else leg(std::false_type{});
    // the block's smoothed values
    {
        const TlRange r = tl_range<S>(p, 0);
        const size_t base = (size_t)p.pj * g.hx + p.hg;
        const int par0 = (p.pj + p.pk0 + 3) & 1;  // red
        const bool ra = par0 ? r.v1 : r.v0, rb_ = par0 ? r.v0 : r.v1;
#pragma unroll
        for (int j = 0; j < S::PZ; j++) {
            const int pk = p.pk0 + j;
            if (pk < r.zlo || pk > r.zhi) continue;
            if ((j & 1) ? ra : rb_) u_out[g.cs + (size_t)pk * g.ps + base] = ub[j];
            if (RULE && ((j & 1) ? rb_ : ra)) u_out[(size_t)pk * g.ps + base] = ur[j];
        }
    }
    __syncthreads();
    // the residuals in natural order over the block, then their means
    {
        const int x0 = 2 * p.hg - p.X0, y = p.pj - p.Y0;
        const int par0 = (p.pj + p.pk0 + 3) & 1;
        const bool yin = p.in_col && y >= 0 && y < TX;
#pragma unroll
        for (int j = 0; j < S::PZ; j++) {
            const int z = p.pk0 + j - p.Z0;
            if (z < 0 || z >= TZ) continue;
            const int xr = x0 + ((j & 1) ? par0 ^ 1 : par0), xb = x0 + ((j & 1) ? par0 : par0 ^ 1);
            C* const row = lds + (z * TX + y) * TX;
            if (yin && xr >= 0 && xr < TX) row[xr] = rr[j];
            if (yin && xb >= 0 && xb < TX) row[xb] = rb[j];
        }
    }
    __syncthreads();
    constexpr int TC2 = TX / 2;
    for (int t = threadIdx.x; t < TC2 * TC2 * (TZ / 2); t += S::NT) {
        const int ci = t % TC2, cj = t / TC2 % TC2, ck = t / (TC2 * TC2);
        const int I = (p.X0 + 1) / 2 + ci, J = (p.Y0 + 1) / 2 + cj, K = (p.Z0 + 1) / 2 + ck;
        if (I > gc.nx - 2 || J > gc.ny - 2 || K > gc.nz - 2) continue;
        const C* const q = lds + ((2 * ck) * TX + 2 * cj) * TX + 2 * ci;
        C sum = (C)0;
#pragma unroll
        for (int dz = 0; dz < 2; dz++)
#pragma unroll
            for (int dy = 0; dy < 2; dy++)
#pragma unroll
                for (int dx = 0; dx < 2; dx++) sum += q[(dz * TX + dy) * TX + dx];
        fc[pos<3, T>(gc, I, J, K)] = (sum * scale);
    }
}

// The up leg: u_in (the down leg's result) plus the interpolated correction ec of
// the coarse level, NPOST sweeps, to u_out (both colours).  Without RULE the
// black points alone are corrected (a red half sweep follows, which reads only
// black ones) and the ghost layer is read from `ring`.  NORM: the max norm of
// the residual of the result into maxbits.
template <typename T, int NPOST, bool RULE, typename S>
__global__ void __launch_bounds__(S::NT)
k_tile_up3(const T* __restrict__ u_in, const T* ring, const T* __restrict__ f, SGrid g, T* u_out,
            T h2, T inv2d, T inv_h2,
            GRule<T> gr, SGrid gc, const T* __restrict__ ec,
            GRule<T> gcr, int nbx, int nby, int rev, unsigned long long* maxbits)
{
    using C = T;
    constexpr bool NORM = !RULE;
    constexpr int H = S::H;
    static_assert(H == 2 * NPOST + NORM, "a halo point per half sweep that follows");
    static_assert(S::PZ % 2 == 0 && S::TZ % 2 == 0, "a thread's planes start at the same parity");
    constexpr int CX = S::HC + 1, CY = S::RY / 2 + 2, CZ = S::RZ / 2 + 2;
    __shared__ __align__(16) C lds[2 * S::CS + CX * CY * CZ];
    if (batch_idle(g)) return;
    u_in = batch_at(u_in, g);
    ring = batch_at(ring, g);
    f = batch_at(f, g);
    u_out = batch_at(u_out, g);
    ec = batch_at(ec, gc);
    if (NORM) maxbits += blockIdx.y;
    C* const R = lds + S::FRONT;
    C* const B = lds + S::CS + S::FRONT;
    C* const E = lds + 2 * S::CS;
    const TlPlace<S> p(g, nbx, nby, rev);
    // coarse values around the region, the rule applied where they are ghosts
    const int cx0 = (p.X0 - H) >> 1, cy0 = (p.Y0 - H) >> 1, cz0 = (p.Z0 - H) >> 1;
    for (int t = threadIdx.x; t < CX * CY * CZ; t += S::NT) {
        const int a = t % CX, b = t / CX % CY, c = t / (CX * CY);
        const AxisNb<C> ax = axis_nb_clamped(max(cx0 + a, 0), gc.nx - 2, gcr, 0);
        const AxisNb<C> ay = axis_nb_clamped(max(cy0 + b, 0), gc.ny - 2, gcr, 1);
        const AxisNb<C> az = axis_nb_clamped(max(cz0 + c, 0), gc.nz - 2, gcr, 2);
        C v = (C)at<3>(ec, gc, ax.q, ay.q, az.q);
        if (ax.ghost) v = ax.fac * v;
        if (ay.ghost) v = ay.fac * v;
        if (az.ghost) v = az.fac * v;
        E[t] = v;
    }
    C fr[S::PZ], fb[S::PZ], ur[S::PZ], ub[S::PZ];
    tl_load<S>(f, g, p, fr, fb);
    const int par0 = (p.pj + p.pk0 + 3) & 1;  // red
    if constexpr (RULE) {
        tl_load<S>(u_in, g, p, ur, ub);
    } else {
        const bool ok = p.in_col && p.hg >= 0 && p.hg < g.hx && p.pj >= 0 && p.pj < g.ny;
        const size_t base = (size_t)p.pj * g.hx + p.hg;
        const bool row_ring = p.pj == 0 || p.pj == g.ny - 1;
#pragma unroll
        for (int j = 0; j < S::PZ; j++) {
            const int pk = p.pk0 + j;
            ur[j] = (C)0;
            ub[j] = (C)0;
            if (p.zl0 + j < S::RZ && pk >= 0 && pk < g.nz && ok) {
                const int xr = 2 * p.hg + ((j & 1) ? par0 ^ 1 : par0), xb = 2 * p.hg + ((j & 1) ? par0 : par0 ^ 1);
                const bool pr = row_ring || pk == 0 || pk == g.nz - 1;
                if (pr || xr == 0 || xr == g.nx - 1) ur[j] = (C)ring[(size_t)pk * g.ps + base];
                if (pr || xb == 0 || xb == g.nx - 1) ub[j] = (C)ring[g.cs + (size_t)pk * g.ps + base];
                else ub[j] = (C)u_in[g.cs + (size_t)pk * g.ps + base];
            }
        }
    }
    __syncthreads();
    {
        // Interpolation: the x parent and neighbour of a column's points are
        // coarse columns h and h + 1, in that order for the even point and
        // the other for the odd one; rows and planes alike.  Per coarse plane the
        // xy interpolants of both points, then along z.
        constexpr int KP = S::PZ / 2 + 2;
        constexpr int zodd = (1 + H) & 1;  // parity of the thread's first plane (block planes start odd, PZ and TZ are even)
        const int ly = p.pj >> 1;
        const int rowp = ly + (p.pj & 1) - cy0, rown = ly + 1 - (p.pj & 1) - cy0;
        const int k0 = (p.pk0 >> 1) - cz0;
        const int c0 = p.hg - cx0;
        C V0[KP], V1[KP];
#pragma unroll
        for (int m = 0; m < KP; m++) {
            const int k = min(k0 + m, CZ - 1);
            const C p0 = E[(k * CY + rowp) * CX + c0], p1 = E[(k * CY + rowp) * CX + c0 + 1];
            const C n0 = E[(k * CY + rown) * CX + c0], n1 = E[(k * CY + rown) * CX + c0 + 1];
            V0[m] = prolong34(prolong34(p0, p1), prolong34(n0, n1));
            V1[m] = prolong34(prolong34(p1, p0), prolong34(n1, n0));
        }
        const TlRange r = tl_range<S>(p, H);
        const bool ra = par0 ? r.v1 : r.v0, rb = par0 ? r.v0 : r.v1;
#pragma unroll
        for (int j = 0; j < S::PZ; j++) {
            const int pk = p.pk0 + j;
            if (p.zl0 + j >= S::RZ) continue;
            const int m = (zodd + j) >> 1;  // (pk >> 1) - (pk0 >> 1)
            const bool odd = (zodd + j) & 1;
            const int mp = odd ? m + 1 : m, mn = odd ? m : m + 1;
            const C e = prolong34(V0[mp], V0[mn]);  // the even point
            const C o = prolong34(V1[mp], V1[mn]);  // the odd point
            const bool zin = pk >= r.zlo && pk <= r.zhi;
            const bool par = (j & 1) ? !par0 : (bool)par0;  // the red point is the odd one
            const bool vr = (j & 1) ? rb : ra, vbk = (j & 1) ? ra : rb;
            if (RULE && zin && vr) ur[j] = (ur[j] + (par ? o : e));
            if (zin && vbk) ub[j] = (ub[j] + (par ? e : o));
        }
    }
    tl_keep<S>(R, B, p, ur, ub);
    __syncthreads();
    unsigned long long best = 0;
    const auto leg = [&](auto edge) {
        constexpr bool Ed = decltype(edge)::value;
#pragma unroll
        for (int it = 0; it < NPOST; it++) {
            tl_sweep<0, RULE, Ed, true, S>(R, B, ur, ub, fr, p, 2 * (NPOST - it) - 1 + NORM, h2, inv2d, gr);
            __syncthreads();
            if (NORM || it + 1 < NPOST) {
                tl_sweep<1, RULE, Ed, true, S>(R, B, ur, ub, fb, p, 2 * (NPOST - it) - 2 + NORM, h2, inv2d, gr);
                __syncthreads();
            } else {
                tl_sweep<1, RULE, Ed, false, S>(R, B, ur, ub, fb, p, 0, h2, inv2d, gr);
            }
        }
        if constexpr (NORM) {
            C rr[S::PZ], rb[S::PZ];
            tl_resid<0, RULE, Ed, S>(R, B, ur, ub, fr, p, inv_h2, gr, rr);
            tl_resid<1, RULE, Ed, S>(R, B, ur, ub, fb, p, inv_h2, gr, rb);
#pragma unroll
            for (int j = 0; j < S::PZ; j++) {
                const unsigned long long a = abs_bits((double)rr[j]), b = abs_bits((double)rb[j]);
                best = max(best, max(a, b));
            }
        }
    };
    if (RULE && p.edge()) leg(std::true_type{});
    else leg(std::false_type{});
    {
        const TlRange r = tl_range<S>(p, 0);
        const size_t base = (size_t)p.pj * g.hx + p.hg;
        const bool ra = par0 ? r.v1 : r.v0, rb = par0 ? r.v0 : r.v1;
#pragma unroll
        for (int j = 0; j < S::PZ; j++) {
            const int pk = p.pk0 + j;
            if (pk < r.zlo || pk > r.zhi) continue;
            if ((j & 1) ? rb : ra) u_out[(size_t)pk * g.ps + base] = ur[j];
            if ((j & 1) ? ra : rb) u_out[g.cs + (size_t)pk * g.ps + base] = ub[j];
        }
    }
    if constexpr (NORM) block_max_to_w<S::NT / 64, true>(best, maxbits);
}

}  // namespace

// ------------------------------------------------------------------ launches
// Block shapes per halo width H (one point per half sweep or residual that follows), G
// ranges of PZ planes each.  The smaller a block, the shorter its chains and the more
// halo per point: 4 x 4 x 4, 8 x 8 x 4, 8 x 8 x 8 or 16 x 16 x 8 points.  Two planes per
// thread where that fits 16 wavefronts.
enum class Form { tiny, flat, small, wide };

template <int H, int TX, int TZ, int PZ>
using TlEven = TlShape<H, TX, TZ, (TZ + 2 * H + PZ - 1) / PZ, PZ>;

template <int H, Form F>
struct TlPick;
template <int H> struct TlPick<H, Form::tiny> { using S = TlEven<H, 4, 4, 2>; };
template <int H> struct TlPick<H, Form::flat> { using S = TlEven<H, 8, 4, (H <= 3 ? 2 : 4)>; };
template <int H> struct TlPick<H, Form::small> { using S = TlEven<H, 8, 8, (H <= 3 ? 2 : 4)>; };
template <> struct TlPick<2, Form::wide> { using S = TlShape<2, 16, 8, 3, 4>; };
template <> struct TlPick<3, Form::wide> { using S = TlShape<3, 16, 8, 4, 4>; };
template <> struct TlPick<4, Form::wide> { using S = TlShape<4, 16, 8, 3, 6>; };
template <> struct TlPick<5, Form::wide> { using S = TlShape<5, 16, 8, 2, 10>; };

static long tl_blocks(const SGrid& g, int tx, int tz)
{
    return (long)ceil_div(g.nx - 2, tx) * ceil_div(g.ny - 2, tx) * ceil_div(g.nz - 2, tz);
}

bool level_legs_fit(int n_pre, int n_post)
{
    return (n_pre == 1 || n_pre == 2) && (n_post == 1 || n_post == 2);
}

// The smallest blocks of which there is at most one per CU; wide ones up to 1024 small blocks'
// worth (256 wide; batch members included).  Beyond that their halo (four to eight times
// the block's work, which idle CUs do for nothing) costs about what streaming does in FP64,
// and more than the per-pass kernels in FP32.  Measured in FP64, the coarse legs of two pre-
// and one post-smoothing sweep (tiny / flat / small / wide), down + up: 17^3 points (125 tiny
// blocks) 6.3 + 4.9 / 8.5 + 5.4 / 8.9 + 5.9 us; 25^3 (343) 8.9 + 5.5 / 8.5 + 5.4 / 9.0 + 6.0;
// 33^3 (225 flat) 12.1 + 6.4 / 8.6 + 5.5 / 9.1 + 6.1 / 13.1 + 8.3; 41^3 (396) - / 15.5 + 7.0 /
// 9.2 + 6.1; and small / wide / streamed / per pass: 33^3 - / - / 22.8 + 13.2 / 31; 49^3 (343
// small) 16.3 + 9.1 / 13.3 + 8.5 / 23.9 + 13.4; 65^3 (729) 23.9 + 13.9 / 13.5 + 8.6 / 23.7 +
// 13.5 / 41; 81^3 (1331) 43 + 21 / 25.5 + 15.1 / 28.2 + 16.6.  FP32 V(1,2): 17^3 4.2 + 6.1 /
// 4.5 + 7.7 / 5.0 + 7.8, 33^3 5.2 + 11.7 / 4.6 + 7.9 / 5.1 + 8.1 / 6.5 + 11.0, 65^3 wide 6.7 +
// 11.9 against 35 per pass, 129^3 20 + 49 (in blocks of 16^3) against 51.
constexpr long kTileBlocks = 1024, kTileCUs = 256;

bool level_tile(int dim, const SGrid& g)
{
    if (dim == 2) return true;
    return tl_blocks(g, 8, 8) * g.nb <= kTileBlocks;
}

// calls go with the form of the level's blocks
template <typename Fn>
static void tl_form(const SGrid& g, Fn go)
{
    if (tl_blocks(g, 4, 4) * g.nb <= kTileCUs) go(std::integral_constant<Form, Form::tiny>{});
    else if (tl_blocks(g, 8, 4) * g.nb <= kTileCUs) go(std::integral_constant<Form, Form::flat>{});
    else if (tl_blocks(g, 8, 8) * g.nb <= kTileCUs) go(std::integral_constant<Form, Form::small>{});
    else go(std::integral_constant<Form, Form::wide>{});
}

template <typename T, int NPRE, bool RULE>
static void down3(hipStream_t st, const LevelLeg& a, const T* u_in, const T* f, T* u_out, T* fc)
{
    tl_form(a.g, [&](auto form) {
        using S = typename TlPick<2 * NPRE + !RULE, decltype(form)::value>::S;
        hipLaunchKernelGGL((k_tile_down3<T, NPRE, RULE, S>), dim3((unsigned)tl_blocks(a.g, S::TX, S::TZ), a.g.nb), dim3(S::NT), 0,
                           st, u_in, f, a.g, u_out, (T)a.h2, (T)(1.0 / 6.0), (T)a.inv_h2, (T)0.125, grule<T>(a.rule), a.gc,
                           fc, ceil_div(a.g.nx - 2, S::TX), ceil_div(a.g.ny - 2, S::TX), a.rev);
    });
}

template <typename T, int NPOST, bool RULE>
static void up3(hipStream_t st, const LevelLeg& a, const T* u_in, const T* ring, const T* f, T* u_out, const T* ec,
                unsigned long long* maxbits)
{
    tl_form(a.g, [&](auto form) {
        using S = typename TlPick<2 * NPOST + !RULE, decltype(form)::value>::S;
        hipLaunchKernelGGL((k_tile_up3<T, NPOST, RULE, S>), dim3((unsigned)tl_blocks(a.g, S::TX, S::TZ), a.g.nb), dim3(S::NT), 0, st,
                           u_in, ring, f, a.g, u_out, (T)a.h2, (T)(1.0 / 6.0), (T)a.inv_h2, grule<T>(a.rule), a.gc, ec,
                           grule<T>(a.coarse_rule), ceil_div(a.g.nx - 2, S::TX), ceil_div(a.g.ny - 2, S::TX), a.rev, maxbits);
    });
}

template <typename T>
void launch_level_down(hipStream_t st, const LevelLeg& a, int n_pre, const T* f, T* u, T* fc)
{
    if (a.dim == 2) return launch_tile2_down<T>(st, a, n_pre, f, u, fc);
    if (!level_tile(3, a.g)) return launch_stream_down<T>(st, a, n_pre, f, u, fc);
    if (n_pre == 1) down3<T, 1, true>(st, a, u, f, u, fc);
    else down3<T, 2, true>(st, a, u, f, u, fc);
}

template <typename T>
void launch_level_up(hipStream_t st, const LevelLeg& a, int n_post, const T* u_in, const T* f, T* u_out, const T* ec)
{
    if (a.dim == 2) return launch_tile2_up<T>(st, a, n_post, u_in, f, u_out, ec);
    if (!level_tile(3, a.g)) return launch_stream_up<T>(st, a, n_post, u_in, f, u_out, ec);
    if (n_post == 1) up3<T, 1, true>(st, a, u_in, u_in, f, u_out, ec, nullptr);
    else up3<T, 2, true>(st, a, u_in, u_in, f, u_out, ec, nullptr);
}

void launch_level0_down(hipStream_t st, const LevelLeg& a, int n_pre, const double* u_in, const double* f, double* u_out,
                        double* fc)
{
    if (a.dim == 2) return launch_tile20_down(st, a, n_pre, u_in, f, u_out, fc);
    if (!level_tile(3, a.g)) return launch_stream0_down(st, a, n_pre, u_in, f, u_out, fc);
    if (n_pre == 1) down3<double, 1, false>(st, a, u_in, f, u_out, fc);
    else down3<double, 2, false>(st, a, u_in, f, u_out, fc);
}

void launch_level0_up(hipStream_t st, const LevelLeg& a, int n_post, const double* u_in, const double* ring,
                      const double* f, double* u_out, const double* ec, unsigned long long* maxbits)
{
    if (a.dim == 2) return launch_tile20_up(st, a, n_post, u_in, ring, f, u_out, ec, maxbits);
    if (!level_tile(3, a.g)) return launch_stream0_up(st, a, n_post, u_in, ring, f, u_out, ec, maxbits);
    if (n_post == 1) up3<double, 1, false>(st, a, u_in, ring, f, u_out, ec, maxbits);
    else up3<double, 2, false>(st, a, u_in, ring, f, u_out, ec, maxbits);
}

template void launch_level_down<double>(hipStream_t, const LevelLeg&, int, const double*, double*, double*);
template void launch_level_down<float>(hipStream_t, const LevelLeg&, int, const float*, float*, float*);
template void launch_level_up<double>(hipStream_t, const LevelLeg&, int, const double*, const double*, double*, const double*);
template void launch_level_up<float>(hipStream_t, const LevelLeg&, int, const float*, const float*, float*, const float*);

}  // namespace np
