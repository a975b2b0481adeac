// Fused V-cycle legs of a 2-D multigrid level (gfx950).
//
// The 2-D levels are bound by launch latency up to about 1000^2 points: a kernel takes
// 3-5 us whether it sweeps 66^2 or 514^2 points, and a V(2,1)
// cycle runs eight of them per level.  As on the small 3-D levels (np_tile.hip) a
// whole leg of the cycle is one launch here:
//   down: the pre-smoothing sweeps, the residual and its restriction;
//   up:   the prolongation and correction, the post-smoothing sweeps and on
//         multigrid level 0 (for the stop test) the residual's max norm.
// A workgroup owns a block of TX x TX points and takes it through every half sweep
// in LDS, with a halo one point wide per half sweep that follows (H in all), which
// it recomputes from arrays that no workgroup of the launch writes.  A thread owns a
// compact column h of a row for both colours; the rows of either colour lie in LDS one
// after the other.  Every operation and its order are those of the per-pass kernels
// (np_kernels.hip), so the iterates are the same bit for bit.
//
// What bounds it: the chain of a load, N half sweeps of an LDS round trip and a
// barrier, and a store: 4 to 5 us a leg up to 514^2 points, with the halo's work 15 us
// at 1026^2; per pass 26 to 30 us a level and cycle, 52 at 1026^2.  On larger levels the points
// decide, and the legs stay ahead of the per-pass kernels: six cycles of a single level, per pass
// and legs, FP64 V(2,1) 2048^2 1.98 / 1.09 ms, 4096^2 4.32 / 3.11, 8192^2 15.0 / 11.2, 16384^2
// (the largest there is) 60.3 / 43.3; V(2,2) 4096^2 5.08 / 3.88; FP32's coarse levels 4096^2
// 3.30 / 2.85, 8192^2 11.5 / 11.4, 16384^2 46 / 45.
#include <type_traits>

#include "np_device.h"

// multiply-adds are written out, as in the other forms of the legs
#pragma clang fp contract(off)

namespace np {

namespace {

// Region of a block of TX x TX points with a halo of H points: HC compact columns per
// row, RY rows, a thread each.
template <int H_, int TX_>
struct T2Shape {
    static constexpr int H = H_, TX = TX_;
    static constexpr int HC = TX / 2 + (H | 1);  // the region starts at an odd x for even H
    static constexpr int RY = TX + 2 * H;
    static constexpr int NCOL = HC * RY;
    static constexpr int NT = (NCOL + 63) / 64 * 64;
    static constexpr int PAD = HC + 1;          // neighbours read beside the region stay in LDS
    static constexpr int CS = NCOL + 2 * PAD;   // LDS elements per colour
    static constexpr int CX = HC + 1, CY = RY / 2 + 2;  // coarse points under the region
    static_assert(NT <= 1024 && TX % 2 == 0, "a thread per compact column");
};

template <typename T>
struct T2Args {
    const T* u_in;  // the state the leg starts from (up: the down leg's result)
    const T* ring;  // up, multigrid level 0: the ghost layer
    const T* f;
    T* u_out;
    T* fc;          // down: coarse right-hand side
    const T* ec;    // up: coarse correction
    SGrid g, gc;
    T h2, inv2d, inv_h2;
    GRule<T> gr, gcr;
    int nbx, rev;
    unsigned long long* maxbits;
};

// N sweeps, up or down.  RULE: a coarse level (ghost values by its rule, the down leg
// starts from zero); otherwise multigrid level 0 (ghost layer in memory, the up leg forms
// the max norm of the residual).
template <typename T, int N, bool RULE, bool UP, typename S>
__global__ void __launch_bounds__(S::NT) k_tile2(T2Args<T> A)
{
    constexpr int H = S::H, TX = S::TX, HC = S::HC;
    constexpr bool ZERO = RULE && !UP, NORM = UP && !RULE;
    static_assert(H == 2 * N + !RULE, "a halo point per half sweep or residual that follows");
    constexpr int EN = UP ? S::CX * S::CY : 0;
    __shared__ __align__(16) T lds[2 * S::CS + EN];
    static_assert(TX * TX <= 2 * S::CS, "the residuals fit in the region's LDS");
    if (batch_idle(A.g)) return;
    const SGrid& g = A.g;
    const SGrid& gc = A.gc;
    T* const B[2] = {lds + S::PAD, lds + S::CS + S::PAD};  // by colour
    const int Nx = g.nx - 2, Ny = g.ny - 2;
    int lb = (int)xcd_block();
    if (A.rev) lb = (int)gridDim.x - 1 - lb;
    const int X0 = 1 + TX * (lb % A.nbx), Y0 = 1 + TX * (lb / A.nbx);
    const int tid = (int)threadIdx.x;
    const bool in_reg = tid < S::NCOL;
    const int t = in_reg ? tid : S::NCOL - 1;
    const int ly = t / HC, lh = t - ly * HC;
    const int hg = ((X0 - H) >> 1) + lh, pj = Y0 - H + ly;
    const bool inside = in_reg && hg >= 0 && hg < g.hx && pj >= 0 && pj < g.ny;
    const size_t row = inside ? (size_t)pj * g.hx + hg : 0;
    const int par0 = pj & 1;  // the red point is x = 2 h + par0, the black one the other
    const int px[2] = {2 * hg + par0, 2 * hg + (par0 ^ 1)};

    // ---- loads
    T fv[2], u[2];
#pragma unroll
    for (int c = 0; c < 2; c++) {
        fv[c] = batch_at(A.f, g)[(c ? g.cs : (size_t)0) + row];
        u[c] = 0;
        if constexpr (!ZERO) {
            const bool ghost = px[c] == 0 || px[c] == g.nx - 1 || pj == 0 || pj == g.ny - 1;
            const T* const src = UP && !RULE && ghost ? batch_at(A.ring, g) : batch_at(A.u_in, g);
            // (up, level 0: the red points are relaxed before they are read)
            if (!UP || RULE || c == 1 || ghost) u[c] = src[(c ? g.cs : (size_t)0) + row];
        }
        if (!inside) fv[c] = u[c] = 0;
    }
    if constexpr (UP) {
        // coarse values around the region, the rule applied where they are ghosts
        T* const E = lds + 2 * S::CS;
        const int cx0 = (X0 - H) >> 1, cy0 = (Y0 - H) >> 1;
        for (int e = tid; e < EN; e += S::NT) {
            const int b = e / S::CX, a = e - b * S::CX;
            const AxisNb<T> ax = axis_nb_clamped(max(cx0 + a, 0), gc.nx - 2, A.gcr, 0);
            const AxisNb<T> ay = axis_nb_clamped(max(cy0 + b, 0), gc.ny - 2, A.gcr, 1);
            T v = at<2>(batch_at(A.ec, gc), gc, ax.q, ay.q, 0);
            if (ax.ghost) v = ax.fac * v;
            if (ay.ghost) v = ay.fac * v;
            E[e] = v;
        }
        __syncthreads();
        // the x parent and neighbour of a column's points are coarse columns h and h + 1 (in
        // that order for the even point, the other for the odd one), rows alike
        const int rp = ((pj >> 1) + (pj & 1) - cy0) * S::CX + lh, rn = ((pj >> 1) + 1 - (pj & 1) - cy0) * S::CX + lh;
        const T p0 = E[rp], p1 = E[rp + 1], n0 = E[rn], n1 = E[rn + 1];
        const T ve = prolong34(prolong34(p0, p1), prolong34(n0, n1)), vo = prolong34(prolong34(p1, p0), prolong34(n1, n0));
#pragma unroll
        for (int c = 0; c < 2; c++) {
            const bool act = inside && px[c] >= 1 && px[c] <= Nx && pj >= 1 && pj <= Ny;
            if (act) u[c] = u[c] + ((par0 ^ c) ? vo : ve);
        }
    }
    // x range and rows of the points within rho of the block
    const auto live = [&](int c, int rho) -> bool {
        return in_reg && pj >= max(1, Y0 - rho) && pj <= min(Ny, Y0 + TX - 1 + rho) && px[c] >= max(1, X0 - rho) &&
               px[c] <= min(Nx, X0 + TX - 1 + rho);
    };
    if constexpr (ZERO) {
        // the first red half sweep from zero needs the right-hand side only
        if (live(0, H)) u[0] = ((T)0 - A.h2 * fv[0]) * A.inv2d;
    }
    if (in_reg) {
        B[0][t] = u[0];
        B[1][t] = u[1];
    }
    __syncthreads();

    // the sum of a point's neighbours; me: its own value
    const auto sum4 = [&](int c, T me) -> T {
        const T* const o = B[c ^ 1] + t;
        const int par = par0 ^ c;
        const T mid = o[0], xo = o[par ? 1 : -1];
        T xm = par ? mid : xo, xp = par ? xo : mid, ym = o[-HC], yp = o[HC];
        if constexpr (RULE) {
            rule_pair(px[c], Nx, me, xm, xp, A.gr, 0);
            rule_pair(pj, Ny, me, ym, yp, A.gr, 1);
        }
        T s = xm + xp;
        s = s + ym;
        return s + yp;
    };
    // own values stay in registers: u[c]
#pragma unroll
    for (int it = 0; it < N; it++)
#pragma unroll
        for (int c = 0; c < 2; c++) {
            if (ZERO && it == 0 && c == 0) continue;
            const T v = fma_t(-A.h2, fv[c], sum4(c, u[c])) * A.inv2d;
            if (live(c, 2 * (N - it) - 1 - c + (!UP || NORM))) {
                u[c] = v;
                B[c][t] = v;
            }
            __syncthreads();
        }
    T* const out = batch_at(A.u_out, g);
#pragma unroll
    for (int c = (UP || RULE) ? 0 : 1; c < 2; c++)
        if (live(c, 0)) out[(c ? g.cs : (size_t)0) + row] = u[c];
    if constexpr (!UP || NORM) {
        T r[2];
#pragma unroll
        for (int c = 0; c < 2; c++) r[c] = fma_t(-A.inv_h2, fma_t((T)-4, u[c], sum4(c, u[c])), fv[c]);
        if constexpr (NORM) {
            unsigned long long best = 0;
#pragma unroll
            for (int c = 0; c < 2; c++)
                if (live(c, 0)) best = max(best, abs_bits((double)r[c]));
            block_max_to_w<S::NT / 64, true>(best, A.maxbits + blockIdx.y);
        } else {
            // the residuals in natural order over the block (zero outside the level), then their means
            __syncthreads();
            const int y = pj - Y0;
#pragma unroll
            for (int c = 0; c < 2; c++) {
                const int x = px[c] - X0;
                if (in_reg && y >= 0 && y < TX && x >= 0 && x < TX) lds[y * TX + x] = live(c, 0) ? r[c] : (T)0;
            }
            __syncthreads();
            constexpr int TC = TX / 2;
            if (tid < TC * TC) {
                const int ci = tid % TC, cj = tid / TC;
                const int I = (X0 + 1) / 2 + ci, J = (Y0 + 1) / 2 + cj;
                const T* const q = lds + 2 * cj * TX + 2 * ci;
                T sum = 0;
                sum += q[0];
                sum += q[1];
                sum += q[TX];
                sum += q[TX + 1];
                if (I <= gc.nx - 2 && J <= gc.ny - 2) batch_at(A.fc, gc)[pos<2, T>(gc, I, J, 0)] = sum * (T)0.25;
            }
        }
    }
}

}  // namespace

// ------------------------------------------------------------------ launches
// Blocks of 16 x 16 points have the shorter barriers and the more workgroups (514^2 points:
// 4.8 and 4.6 us a leg against 7.7 and 5.2 in blocks of 32 x 32; 1026^2 down 14.8 against
// 16.8).  Only the legs that end in a maximum over the level take the larger ones where
// the small ones are many: their atomics on one word, 6 ns each, are in a row
// (1026^2: 26 us in 4225 small blocks, 15 in 1089 large ones; 512^2: 10 in 1024, 7 in 256;
// 256^2: 5.9 in 256 small ones).
constexpr long kTile2NormBlocks = 512;

template <typename T, int N, bool RULE, bool UP>
static void tile2(hipStream_t st, T2Args<T> A)
{
    constexpr int H = 2 * N + !RULE;
    const auto go = [&](auto s) {
        using S = decltype(s);
        A.nbx = ceil_div(A.g.nx - 2, S::TX);
        hipLaunchKernelGGL((k_tile2<T, N, RULE, UP, S>), dim3((unsigned)(A.nbx * ceil_div(A.g.ny - 2, S::TX)), A.g.nb),
                           dim3(S::NT), 0, st, A);
    };
    const long small = (long)ceil_div(A.g.nx - 2, 16) * ceil_div(A.g.ny - 2, 16) * A.g.nb;
    if constexpr (UP && !RULE) {
        if (small > kTile2NormBlocks) return go(T2Shape<H, 32>{});
    }
    go(T2Shape<H, 16>{});
}

template <typename T>
static T2Args<T> tile2_args(const LevelLeg& a, const T* u_in, const T* ring, const T* f, T* u_out, T* fc, const T* ec,
                            unsigned long long* maxbits)
{
    T2Args<T> A{};
    A.u_in = u_in;
    A.ring = ring;
    A.f = f;
    A.u_out = u_out;
    A.fc = fc;
    A.ec = ec;
    A.g = a.g;
    A.gc = a.gc;
    A.h2 = (T)a.h2;
    A.inv2d = (T)(1.0 / 4.0);
    A.inv_h2 = (T)a.inv_h2;
    A.gr = grule<T>(a.rule);
    A.gcr = grule<T>(a.coarse_rule);
    A.rev = a.rev;
    A.maxbits = maxbits;
    return A;
}

template <typename T>
void launch_tile2_down(hipStream_t st, const LevelLeg& a, int n_pre, const T* f, T* u, T* fc)
{
    const T2Args<T> A = tile2_args<T>(a, u, u, f, u, fc, nullptr, nullptr);
    if (n_pre == 1) tile2<T, 1, true, false>(st, A);
    else tile2<T, 2, true, false>(st, A);
}

template <typename T>
void launch_tile2_up(hipStream_t st, const LevelLeg& a, int n_post, const T* u_in, const T* f, T* u_out, const T* ec)
{
    const T2Args<T> A = tile2_args<T>(a, u_in, u_in, f, u_out, nullptr, ec, nullptr);
    if (n_post == 1) tile2<T, 1, true, true>(st, A);
    else tile2<T, 2, true, true>(st, A);
}

void launch_tile20_down(hipStream_t st, const LevelLeg& a, int n_pre, const double* u_in, const double* f, double* u_out,
                        double* fc)
{
    const T2Args<double> A = tile2_args<double>(a, u_in, u_in, f, u_out, fc, nullptr, nullptr);
    if (n_pre == 1) tile2<double, 1, false, false>(st, A);
    else tile2<double, 2, false, false>(st, A);
}

void launch_tile20_up(hipStream_t st, const LevelLeg& a, int n_post, const double* u_in, const double* ring,
                      const double* f, double* u_out, const double* ec, unsigned long long* maxbits)
{
    const T2Args<double> A = tile2_args<double>(a, u_in, ring, f, u_out, nullptr, ec, maxbits);
    if (n_post == 1) tile2<double, 1, false, true>(st, A);
    else tile2<double, 2, false, true>(st, A);
}

template void launch_tile2_down<double>(hipStream_t, const LevelLeg&, int, const double*, double*, double*);
template void launch_tile2_down<float>(hipStream_t, const LevelLeg&, int, const float*, float*, float*);
template void launch_tile2_up<double>(hipStream_t, const LevelLeg&, int, const double*, const double*, double*, const double*);
template void launch_tile2_up<float>(hipStream_t, const LevelLeg&, int, const float*, const float*, float*, const float*);

}  // namespace np
