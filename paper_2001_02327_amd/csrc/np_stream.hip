// Fused V-cycle legs of a large 3-D multigrid level (gfx950): FP64, and the largest coarse
// levels in FP32.
//
// A V(2,1) cycle in kernels that each make one pass over the level moves 89 B per
// point in FP64, where 36 B would do.  Here a whole leg of the cycle is one launch:
//   down: the pre-smoothing sweeps, the residual and its restriction;
//   up:   the prolongation and correction, the post-smoothing sweeps and on
//         multigrid level 0 (for the stop test) the residual's max norm.
//
// A workgroup owns a column of TX x TY points and a chunk of planes.  It marches
// up in z with every half sweep of the leg in flight at once: in the step of
// plane a the first red half sweep works on plane a, the first black one on
// plane a - 1, the second red one on plane a - 2 and so on, the residual behind
// the last.  A point's z-neighbours are then values its own thread holds in
// registers (one of them formed a moment ago), its x- and y-neighbours were put
// into LDS by other threads in the step before: each value is loaded from
// memory once and stored once, and one barrier per plane orders everything.
// Around its column a workgroup recomputes a halo of H points (one per half
// sweep that follows), whose values it reads from arrays that no workgroup of the
// launch writes, so the result does not depend on the order of the workgroups.
//
// A thread owns the compact column h of two neighbouring rows for both colours (the
// rows are each other's y-neighbours: four LDS reads per stage instead of six, and
// twice the independent work to hide LDS latency behind).  In the step of plane a
// every stage's point of a column has the same x = 2 h + par (colour and plane
// alternate together), hence one mask and one x-neighbour offset per step, which
// are known where the step is compiled.  Every operation and its order are those
// of the per-pass kernels (np_kernels.hip), so the iterates are the same bit for
// bit.
//
// What bounds it: a step is some 200 instructions per wavefront, 25 LDS accesses and a
// barrier, with the registers of two wavefronts per SIMD in FP64: 1.2 to 1.4 us, and the
// columns along the boundary, whose steps are the longest, decide; at 514^3 points the
// memory system as much: 2.9 and 3.5 GB moved a leg, a third of the reads the halo's that the
// L2 did not keep, at 4.0 and 4.2 TB/s (2.3 and 2.85 GB that a leg cannot do without: 3.2
// and 3.5 TB/s; non-temporal stores do not help: 758 and 871 us).
// Measured, V(2,1) in FP64, down + up: 514^3 729 + 816 us against 2.79 ms in full sweeps,
// restriction and prolongation; 258^3 107 + 114 us against 419; 130^3 32 + 26 against 87; coarse 129^3 35 + 22 against 80.
// FP32, two workgroups per CU: coarse 257^3 67 + 60 us against 184.
#include <algorithm>
#include <type_traits>

#include "np_device.h"

// Every multiply-add here is written out: the stages of a step hand values to each
// other in registers, and contracted by the compiler a stage's last product would
// reach the next stage's sum unrounded.
#pragma clang fp contract(off)

namespace np {

namespace {

// Region of a column of TX x TY points with a halo of H points: HC compact columns
// per row, RY rows, one thread per compact column of two neighbouring rows.
template <int H_, int TX_, int TY_>
struct LegShape {
    static constexpr int H = H_, TX = TX_, TY = TY_;
    static constexpr int HC = TX / 2 + (H | 1);  // the region starts at an odd x for even H
    static constexpr int RY = TY + 2 * H;
    static constexpr int NCOL = HC * RY;
    static constexpr int NTH = NCOL / 2;         // threads with work
    static constexpr int NT = (NTH + 63) / 64 * 64;
    static constexpr int PAD = HC + 1;           // a neighbour read beside the region stays in LDS
    static constexpr int CX = HC + 1, CY = RY / 2 + 2;  // coarse points under the region
    static_assert(HC == 32 && NT == NTH && RY % 2 == 0, "whole rows per wavefront, two rows per thread");
};

template <typename T>
struct LegArgs {
    const T* u_in;  // the state the leg starts from (up: the down leg's result)
    const T* ring;  // up, multigrid level 0: the ghost layer
    const T* f;
    T* u_out;
    T* fc;          // down: coarse right-hand side
    const T* ec;    // up: coarse correction
    SGrid g, gc;
    T h2, inv2d, inv_h2, scale;
    GRule<T> gr, gcr;
    int nbx, nby, kz;  // columns along x and y, planes per chunk
    int rev;
    unsigned long long* maxbits;
};

// One plane of an array as a buffer: accesses past its `bytes` (inactive lanes get such an
// offset, planes without work no bytes at all) read zero and write nothing, so a step
// issues the same loads and stores whatever it does and they can stay in flight for
// several steps (behind branches the compiler has to wait as if none was issued).
constexpr unsigned kLegOob = 0x80000000u;

template <typename T>
__device__ __forceinline__ __amdgpu_buffer_rsrc_t leg_plane(const T* p, bool on, unsigned bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc((void*)p, 0, on ? (int)bytes : 0, 0x00027000);
}

template <typename T>
__device__ __forceinline__ T leg_load(__amdgpu_buffer_rsrc_t b, unsigned off)
{
    if constexpr (sizeof(T) == 8) return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(b, off, 0, 0));
    else return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(b, off, 0, 0));
}

// rule_pair without branches; ql: the index for the test of the lower wall
template <typename C>
__device__ __forceinline__ void leg_rule(int ql, int q, int N, C self, C& lo, C& hi, const GRule<C>& gr, int ax)
{
    lo = ql == 1 ? -self : lo;
    const C up = (gr.xn1[ax] ? (C)-1 : gr.coef[ax]) * (gr.xn1[ax] ? lo : self);
    hi = q == N ? up : hi;
}

// m ? a : b without a branch around what forms a (the compiler made one of every select
// in the steps beside a boundary, which took half as long again as the others)
template <typename T>
__device__ __forceinline__ T leg_select(bool m, T a, T b)
{
    asm volatile("" : "+v"(a));
    return m ? a : b;
}

typedef unsigned LegV2 __attribute__((ext_vector_type(2)));

template <typename T>
__device__ __forceinline__ void leg_store(__amdgpu_buffer_rsrc_t b, unsigned off, T v)
{
    if constexpr (sizeof(T) == 8) __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(LegV2, v), b, off, 0, 0);
    else __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned, v), b, off, 0, 0);
}

constexpr int kLegRule = 0, kLegWarm = 1, kLegZero = 2;

// N sweeps, up or down.  kLegRule: a coarse level (ghost values by its rule, the down leg
// starts from zero); otherwise multigrid level 0 with its ghost layer in memory: kLegWarm from
// u_in, the up leg in FP64 with the max norm of the residual, kLegZero from zero.
template <typename T, int N, int MODE, bool UP, typename S>
__global__ void __launch_bounds__(S::NT, sizeof(T) == 8 ? 2 : 4) k_leg3(LegArgs<T> A)
{
    using C = T;
    constexpr bool RULE = MODE == kLegRule, ZERO = MODE != kLegWarm && !UP, NORM = UP && !RULE && sizeof(T) == 8;
    constexpr bool RES = !UP || NORM;
    constexpr int NX = 2 * N;                          // half sweeps
    constexpr int NA = (ZERO ? 0 : 1) + NX - (RES ? 0 : 1);  // planes other threads read: the start, each half sweep
    constexpr int X0A = ZERO ? 0 : 1;                  // LDS plane of the first half sweep
    constexpr int PL = S::NCOL;
    static_assert(S::H == (UP ? NX + NORM : NX + !ZERO), "a halo point per half sweep that follows");
    constexpr int RESN = UP ? 0 : S::TX * S::TY, EN = UP ? S::CX * S::CY : 0;
    __shared__ __align__(16) C lds[2 * NA * PL + 2 * S::PAD + 2 * RESN + 2 * EN];
    if (batch_idle(A.g)) return;
    const SGrid& g = A.g;
    const C* const u_in = batch_at(A.u_in, g);
    const C* const ring = batch_at(A.ring, g);
    const C* const f = batch_at(A.f, g);
    C* const u_out = batch_at(A.u_out, g);
    // plane i of parity s at pl + (2 i + s) PL: the threads' first rows, then their second
    // ones, so that a wavefront reads consecutive elements (a row after the other as in
    // the region, with two rows per thread, two in five LDS cycles went to bank conflicts)
    C* const pl = lds + S::PAD;
    C* const resl = lds + 2 * NA * PL + 2 * S::PAD;
    C* const el = resl + 2 * RESN;
    const int Nx = g.nx - 2, Ny = g.ny - 2, Nz = g.nz - 2;

    int lb = (int)xcd_block();
    if (A.rev) lb = (int)gridDim.x - 1 - lb;
    const int bx = lb % A.nbx, by = lb / A.nbx % A.nby, bz = lb / (A.nbx * A.nby);
    const int X0 = 1 + S::TX * bx, Y0 = 1 + S::TY * by, Z0 = 1 + A.kz * bz;
    // last plane of the chunk; the down leg also forms plane N_z + 1 of an odd N_z
    // (residual zero), the second child plane of the last coarse one
    const int Z1 = min(Z0 + A.kz - 1, Nz), ZE = UP ? Z1 : min(Z0 + A.kz - 1, (Nz + 1) & ~1);
    const int tid = (int)threadIdx.x;
    const int t = min(tid, S::NTH - 1);
    const bool in_reg = tid < S::NTH;
    const int lm = t / S::HC, lh = t - lm * S::HC;
    const int hs = (X0 - S::H) >> 1, ys = Y0 - S::H;
    const int hg = hs + lh, pj = ys + 2 * lm;
    // per row: byte offset in a plane; activity of the even and the odd point; byte offsets of
    // those that the block stores
    unsigned off[2], so0[2], so1[2];
    bool act0[2], act1[2];
#pragma unroll
    for (int r = 0; r < 2; r++) {
        const int y = pj + r;
        const bool inside = hg >= 0 && hg < g.hx && y >= 0 && y < g.ny;
        off[r] = inside ? (unsigned)(y * g.hx + hg) * (unsigned)sizeof(C) : kLegOob;
        const bool yact = inside && y >= 1 && y <= Ny;
        act0[r] = yact && 2 * hg >= 1 && 2 * hg <= Nx;
        act1[r] = yact && 2 * hg + 1 <= Nx;
        const bool yown = in_reg && y >= Y0 && y < Y0 + S::TY;
        so0[r] = act0[r] && yown && 2 * hg >= X0 && 2 * hg < X0 + S::TX ? off[r] : kLegOob;
        so1[r] = act1[r] && yown && 2 * hg + 1 >= X0 && 2 * hg + 1 < X0 + S::TX ? off[r] : kLegOob;
    }
    // a wavefront holds a point beside a wall
    const bool wall_x = __any(2 * hg <= 1 || 2 * hg + 1 >= Nx), wall_y = __any(pj <= 1 || pj + 1 >= Ny);
    const unsigned pbytes = (unsigned)(g.ps * sizeof(C));
    // every block starts at odd coordinates and steps alternate in parity, so the parity of
    // a point is known where the step is compiled: x = 2 h + par in the first row
    constexpr int kStepPar = UP ? NORM : 1;  // parity of the first step's plane
    static_assert(S::TX % 2 == 0 && S::TY % 2 == 0, "blocks start at odd coordinates");
    // the region reaches the boundary in x or y: masks and ghost rules apply
    const bool edge = hs < 1 || ys < 2 || 2 * (hs + S::HC) >= Nx || ys + S::RY > Ny;

    // ---- up: interpolation of the correction.  The x parent and neighbour of a
    // column's points are the coarse columns h and h + 1 (in that order for the even
    // point, the other for the odd one), rows and planes alike.  v0/v1: xy
    // interpolants of the even and the odd point of a row on coarse planes K (c) and K + 1 (n).
    const int cx0 = hs, cy0 = ys >> 1;
    C v0c[2] = {}, v1c[2] = {}, v0n[2] = {}, v1n[2] = {};
    constexpr int NE = UP ? (EN + S::NT - 1) / S::NT : 1;  // coarse points per thread
    // coarse planes in flight and the ghost factors of a thread's points along x and y
    C epf[2][NE] = {};
    C efx[NE], efy[NE];
    unsigned eoff[NE];  // offset in a coarse plane of either colour
    int ecol[NE];       // parity of x + y
    const SGrid& gc = A.gc;
    if constexpr (UP) {
#pragma unroll
        for (int k = 0; k < NE; k++) {
            const int e = min(tid + k * S::NT, EN - 1);
            const int a = e % S::CX, b = e / S::CX;
            const AxisNb<C> ax = axis_nb_clamped(max(cx0 + a, 0), gc.nx - 2, A.gcr, 0);
            const AxisNb<C> ay = axis_nb_clamped(max(cy0 + b, 0), gc.ny - 2, A.gcr, 1);
            efx[k] = ax.ghost ? ax.fac : (C)1;
            efy[k] = ay.ghost ? ay.fac : (C)1;
            eoff[k] = (unsigned)(ay.q * gc.hx + (ax.q >> 1));
            ecol[k] = (ax.q + ay.q) & 1;
        }
    }
    const auto load_e = [&](int K, C (&v)[NE]) {
        if constexpr (UP) {
            const AxisNb<C> az = axis_nb_clamped(max(K, 0), gc.nz - 2, A.gcr, 2);
            const C* const pz = batch_at(A.ec, gc) + (size_t)az.q * gc.ps;
#pragma unroll
            for (int k = 0; k < NE; k++) v[k] = pz[(((ecol[k] + az.q) & 1) ? (size_t)0 : gc.cs) + eoff[k]];
        }
    };
    const auto store_e = [&](int K, const C (&v)[NE]) {
        if constexpr (UP) {
            const AxisNb<C> az = axis_nb_clamped(max(K, 0), gc.nz - 2, A.gcr, 2);
            const C fz = az.ghost ? az.fac : (C)1;
#pragma unroll
            for (int k = 0; k < NE; k++)
                if (tid + k * S::NT < EN) el[(K & 1) * EN + tid + k * S::NT] = fz * (efy[k] * (efx[k] * v[k]));
        }
    };
    const auto interp_e = [&](int K, C (&v0)[2], C (&v1)[2]) {
        if constexpr (UP) {
            const C* const e = el + (K & 1) * EN + (hg - cx0);
#pragma unroll
            for (int r = 0; r < 2; r++) {
                const int y = pj + r;
                const int rp = (y >> 1) + (y & 1) - cy0, rn = (y >> 1) + 1 - (y & 1) - cy0;
                const C p0 = e[rp * S::CX], p1 = e[rp * S::CX + 1], n0 = e[rn * S::CX], n1 = e[rn * S::CX + 1];
                v0[r] = prolong34(prolong34(p0, p1), prolong34(n0, n1));
                v1[r] = prolong34(prolong34(p1, p0), prolong34(n1, n0));
            }
        }
    };

    // ---- memory: what step a takes in (right-hand sides of plane a, the start's black points
    // of plane a + 1, red ones of plane a where something needs them), loaded LEAD steps
    // ahead.  Up, multigrid level 0: the ghost layer comes from `ring`
    constexpr bool RING = UP && !RULE;
    struct Feed {
        C fr[2], fb[2], b[2], r[2], gb[2];
    };
    unsigned offi[2][2], offg[2][2];  // level 0, up: own points and ghost points by parity of x
    if constexpr (RING) {
#pragma unroll
        for (int r = 0; r < 2; r++) {
            offi[r][0] = act0[r] ? off[r] : kLegOob;
            offi[r][1] = act1[r] ? off[r] : kLegOob;
            offg[r][0] = act0[r] ? kLegOob : off[r];
            offg[r][1] = act1[r] ? kLegOob : off[r];
        }
    }
    const auto load = [&](auto par_tag, Feed& q, int a) {
        constexpr int par = decltype(par_tag)::value;  // of x in the first row
        const bool on = a >= 0 && a < g.nz, onb = a + 1 >= 0 && a + 1 < g.nz;
        const C* const fz = f + (ptrdiff_t)a * (ptrdiff_t)g.ps;
        const auto br = leg_plane(fz, on, pbytes), bb = leg_plane(fz + g.cs, on, pbytes);
#pragma unroll
        for (int r = 0; r < 2; r++) {
            q.fr[r] = leg_load<C>(br, off[r]);
            q.fb[r] = leg_load<C>(bb, off[r]);
        }
        if constexpr (!ZERO) {
            const ptrdiff_t pb = (ptrdiff_t)(a + 1) * (ptrdiff_t)g.ps + (ptrdiff_t)g.cs;
            const bool redge = edge || a <= 1 || a >= Nz;
            const auto rr = leg_plane((RING ? ring : u_in) + (ptrdiff_t)a * (ptrdiff_t)g.ps, on && redge, pbytes);
            const bool inz = a + 1 >= 1 && a + 1 <= Nz;
            const auto ub = leg_plane(u_in + pb, RING ? inz : onb, pbytes);
            const auto gb = leg_plane(ring + pb, RING && onb && redge, pbytes);
#pragma unroll
            for (int r = 0; r < 2; r++) {
                const int od = r ? !par : par;
                q.b[r] = leg_load<C>(ub, RING ? offi[r][od] : off[r]);
                q.r[r] = leg_load<C>(rr, off[r]);
                if constexpr (RING) q.gb[r] = leg_load<C>(gb, inz ? offg[r][od] : off[r]);
            }
        }
    };

    // ---- pipeline state, per row.  b0: the start's black points on planes a - 1, a (and a + 1
    // in a step); x1[i], x2[i]: half sweep i's values on planes p - 1, p - 2 for its plane p = a - i
    C b0m[2] = {}, b0c[2] = {};
    C x1[NX][2] = {}, x2[NX][2] = {};
    C frh[NX + 1][2] = {}, fbh[NX][2] = {};  // right-hand sides: red of planes a - i, black of planes a - 1 - i
    C rbh[2] = {};   // residual of the last black half sweep's plane, one step old
    C ered[2] = {};  // up with RULE: the correction of the red point of the next plane
    C rsum = 0;      // down: a coarse point's sum
    unsigned long long best = 0;
    constexpr int CTX = S::TX / 2, NCT = CTX * (S::TY / 2);
    static_assert(UP || NCT <= S::NT, "a thread per coarse point");
    // down: residuals of the block by child (first or second along x and along y), each
    // CTX x TY / 2 values in the order of the coarse points: where the odd point of a
    // row goes (the even one is the coarse point's before, second child)
    int rwo[2];
    bool rw1[2], rw2[2];
#pragma unroll
    for (int r = 0; r < 2; r++) {
        const int y = pj + r - Y0, kb = hg - ((X0 - 1) >> 1);
        const bool yin = in_reg && y >= 0 && y < S::TY;
        rwo[r] = 2 * ((S::H + r) & 1) * NCT + (y >> 1) * CTX + kb;
        rw1[r] = yin && kb >= 0 && kb < CTX;
        rw2[r] = yin && kb >= 1 && kb <= CTX;
    }
    // down: a thread's coarse point, by parity of its x + y
    const unsigned cbytes = (unsigned)(gc.ps * sizeof(C));
    unsigned coff0 = kLegOob, coff1 = kLegOob;
    if constexpr (!UP) {
        const int I = (X0 + 1) / 2 + tid % CTX, J = (Y0 + 1) / 2 + tid / CTX;
        if (tid < NCT && I <= gc.nx - 2 && J <= gc.ny - 2)
            (((I + J) & 1) ? coff1 : coff0) = (unsigned)(J * gc.hx + (I >> 1)) * (unsigned)sizeof(C);
    }

    const auto step = [&](auto edge_tag, auto par_tag, int a, const Feed& q, C (&ep)[NE]) {
        // 0: every point of the step is inside the level; 1: in x and y some are not; 2: nor in z
        constexpr int E = decltype(edge_tag)::value;
        // x = 2 hg + par for every stage of this step in the first row, the other point in the second
        constexpr int par = decltype(par_tag)::value;
        constexpr int pa1 = (par + S::H) & 1;  // parity of a
        constexpr int dx = par ? 1 : -1;
        // (tests against a wall are formed in each step: kept as masks they are more than the
        // scalar registers hold)
        int Nx_ = Nx, Ny_ = Ny;
        asm volatile("" : "+s"(Nx_), "+s"(Ny_));
        bool mx[2];
        unsigned so[2], soo[2];
        int pi[2];
#pragma unroll
        for (int r = 0; r < 2; r++) {
            const bool od = r ? !par : par;
            mx[r] = od ? act1[r] : act0[r];
            so[r] = od ? so1[r] : so0[r];
            soo[r] = od ? so0[r] : so1[r];
            pi[r] = 2 * hg + (od ? 1 : 0);
        }
        // LDS planes of a's parity and of the other one.  Half sweep i reads its source's
        // plane a - i and writes its own plane a - i, each array holding one plane of
        // either parity: what is read in a step is not written in it
        C* const pa = pl + pa1 * PL + t;
        C* const pb = pl + (pa1 ^ 1) * PL + t;
        // ---- every LDS read of the step, before anything waits for one: per stage the other
        // x-neighbour of either row, the row below the first and the row above the second (the
        // rows are each other's y-neighbours).  Stage NX is the red residual
        constexpr int NS = NX + (RES ? 1 : 0);
        C lx[NS][2], ly[NS], lz[NS];
#pragma unroll
        for (int i = ZERO ? 1 : 0; i < NS; i++) {
            const C* const P = ((i & 1) ? pb : pa) + (i == 0 ? 0 : 2 * (X0A + i - 1)) * PL;
            const C (&c)[2] = i == 0 ? b0c : x1[i > 0 ? i - 1 : 0];
            lx[i][0] = dx > 0 ? dpp_next(c[0]) : dpp_prev(c[0]);
            lx[i][1] = dx > 0 ? dpp_prev(c[1]) : dpp_next(c[1]);
            ly[i] = P[S::NTH - S::HC];
            lz[i] = P[S::HC];
        }
        C rch[4];
        const int pp = a - NX - 1;  // down: the plane whose residuals were completed in the step before
        if constexpr (!UP) {
            const C* const rp = resl + (pa1 ^ 1) * RESN + (tid < NCT ? tid : 0);
#pragma unroll
            for (int e = 0; e < 4; e++) rch[e] = rp[e * NCT];
        }
#pragma unroll
        for (int r = 0; r < 2; r++) {
#pragma unroll
            for (int i = NX; i > 0; i--) frh[i][r] = frh[i - 1][r];
            frh[0][r] = q.fr[r];
        }
        // ---- the start's black points of plane a + 1
        C b0p[2] = {}, red0[2] = {};
        if constexpr (!ZERO) {
            const int z = a + 1;
            if constexpr (UP) {
                if constexpr (pa1) {
#pragma unroll
                    for (int r = 0; r < 2; r++) {
                        v0c[r] = v0n[r];
                        v1c[r] = v1n[r];
                    }
                    interp_e((z >> 1) + 1, v0n, v1n);
                } else {
                    store_e((z >> 1) + 2, ep);
                    load_e((z >> 1) + 4, ep);
                }
            }
#pragma unroll
            for (int r = 0; r < 2; r++) {
                b0p[r] = q.b[r];
                if constexpr (UP) {
                    const bool od = r ? !par : par;
                    const C vc = od ? v1c[r] : v0c[r], vn = od ? v1n[r] : v0n[r];
                    const C e = pa1 ? prolong34(vc, vn) : prolong34(vn, vc);
                    b0p[r] = b0p[r] + e;
                    if constexpr (E && !RULE) b0p[r] = leg_select(mx[r] && (E == 1 || (z >= 1 && z <= Nz)), b0p[r], q.gb[r]);
                    if constexpr (E && RULE) {
                        // the start's red point of plane a (the first half sweep's ghost values need it)
                        red0[r] = (q.r[r] + ered[r]);
                        const C wc = od ? v0c[r] : v1c[r], wn = od ? v0n[r] : v1n[r];
                        ered[r] = pa1 ? prolong34(wc, wn) : prolong34(wn, wc);
                    }
                }
            }
        }
        // the sum of each row's point's neighbours on plane p: own column zm, c, zp; me: the points' own values
        const auto sum6 = [&](int i, const C (&zm)[2], const C (&c)[2], const C (&zp)[2], const C (&me)[2], int p, C (&s)[2]) {
            C xm[2], xp[2], y0[2], y1[2], z0[2], z1[2];
#pragma unroll
            for (int r = 0; r < 2; r++) {
                const bool od = r ? !par : par;
                xm[r] = od || !(E && RULE) ? c[r] : lx[i][r];
                xp[r] = od || !(E && RULE) ? lx[i][r] : c[r];
                y0[r] = r ? c[0] : ly[i];
                y1[r] = r ? lz[i] : c[1];
                z0[r] = zm[r];
                z1[r] = zp[r];
            }
            if constexpr (E && RULE) {
                // by wavefront: many hold no point beside a wall (the lower ones are odd)
                if (wall_x) {
#pragma unroll
                    for (int r = 0; r < 2; r++) leg_rule((r ? !par : par) ? pi[r] : 0, pi[r], Nx_, me[r], xm[r], xp[r], A.gr, 0);
                }
                if (wall_y) {
#pragma unroll
                    for (int r = 0; r < 2; r++)
                        leg_rule(((1 + S::H + r) & 1) ? pj + r : 0, pj + r, Ny_, me[r], y0[r], y1[r], A.gr, 1);
                }
                if (E == 2 && (p == 1 || p == Nz)) {
#pragma unroll
                    for (int r = 0; r < 2; r++) leg_rule(p, p, Nz, me[r], z0[r], z1[r], A.gr, 2);
                }
            }
#pragma unroll
            for (int r = 0; r < 2; r++) {
                s[r] = xm[r] + xp[r];
                s[r] = s[r] + y0[r];
                s[r] = s[r] + y1[r];
                s[r] = s[r] + z0[r];
                s[r] = s[r] + z1[r];
            }
        };
        // ---- half sweeps
        C xn[NX][2], sb[2] = {};
#pragma unroll
        for (int i = 0; i < NX; i++) {
            const int p = a - i;
            const bool zin = p >= 1 && p <= Nz;
            if (ZERO && i == 0) {
#pragma unroll
                for (int r = 0; r < 2; r++) {
                    xn[0][r] = ((C)0 - A.h2 * frh[0][r]) * A.inv2d;
                    if constexpr (E && !RULE) xn[0][r] = leg_select(mx[r] && (E == 1 || zin), xn[0][r], (C)0);
                }
                continue;
            }
            // own column of the source: planes p - 1, p, p + 1; old: the points' values before
            const C (&zm)[2] = i == 0 ? b0m : x2[i > 0 ? i - 1 : 0];
            const C (&c)[2] = i == 0 ? b0c : x1[i > 0 ? i - 1 : 0];
            const C (&zp)[2] = i == 0 ? b0p : xn[i > 0 ? i - 1 : 0];
            const C (&old)[2] = i >= 2 ? x2[i >= 2 ? i - 2 : 0] : (i == 1 ? b0m : red0);
            C s[2];
            sum6(i, zm, c, zp, old, p, s);
#pragma unroll
            for (int r = 0; r < 2; r++) {
                const C fv = (i & 1) ? fbh[i > 0 ? i - 1 : 0][r] : frh[i][r];
                C v = fma_t(-A.h2, fv, s[r]) * A.inv2d;
                // (with a rule what stands outside the level is read by no point inside)
                if constexpr (E && !RULE) v = leg_select(mx[r] && (E == 1 || zin), v, i == 0 ? q.r[r] : old[r]);
                xn[i][r] = v;
            }
            if (i == NX - 1 && RES) {
                // the residual of the black points just relaxed
                C s2[2] = {s[0], s[1]};
                if constexpr (E && RULE) sum6(i, zm, c, zp, xn[i], p, s2);
#pragma unroll
                for (int r = 0; r < 2; r++) {
                    const C fv = fbh[NX - 2][r];
                    sb[r] = fma_t(-A.inv_h2, fma_t((C)-6, xn[i][r], s2[r]), fv);
                    if constexpr (E && !UP) sb[r] = leg_select(mx[r] && (E == 1 || zin), sb[r], (C)0);
                }
            }
        }
        // ---- the residual of the red points, plane a - NX
        C rr[2] = {};
        if constexpr (RES) {
            const int p = a - NX;
            const bool zin = p >= 1 && p <= Nz;
            C s[2];
            sum6(NX, x2[NX - 1], x1[NX - 1], xn[NX - 1], x2[NX - 2], p, s);
#pragma unroll
            for (int r = 0; r < 2; r++) {
                rr[r] = fma_t(-A.inv_h2, fma_t((C)-6, x2[NX - 2][r], s[r]), frh[NX][r]);
                if constexpr (E && !UP) rr[r] = leg_select(mx[r] && (E == 1 || zin), rr[r], (C)0);
                if constexpr (UP) {
                    if (p >= Z0 && p <= Z1) {
                        if (so[r] != kLegOob) best = max(best, abs_bits((double)rr[r]));
                        if (soo[r] != kLegOob) best = max(best, abs_bits((double)rbh[r]));
                    }
                }
            }
        }
        // ---- LDS writes of the step
#pragma unroll
        for (int r = 0; r < 2; r++) {
            if constexpr (!ZERO) pb[r * S::NTH] = b0p[r];
#pragma unroll
            for (int i = 0; i < NX; i++)
                if (i < NX - 1 || RES) ((i & 1) ? pb : pa)[2 * (X0A + i) * PL + r * S::NTH] = xn[i][r];
        }
        // ---- results: the black points after the last half sweep, the red ones before it
#pragma unroll
        for (int i = UP || RULE ? NX - 2 : NX - 1; i < NX; i++) {
            const int p = a - i;
            const auto o = leg_plane(u_out + ((i & 1) ? (ptrdiff_t)g.cs : 0) + (ptrdiff_t)p * (ptrdiff_t)g.ps,
                                     p >= Z0 && p <= Z1, pbytes);
#pragma unroll
            for (int r = 0; r < 2; r++) leg_store(o, so[r], xn[i][r]);
        }
        if constexpr (!UP) {
            // a coarse point's children, plane by plane
            constexpr bool odd = (NX + 1 + pa1) & 1;  // plane pp
            if (odd) rsum = (C)0;
            rsum += rch[0];
            rsum += rch[1];
            rsum += rch[2];
            rsum += rch[3];
            if constexpr (!odd) {
                const int K = pp >> 1;
                const bool on = pp >= Z0 && pp <= ZE && K <= gc.nz - 2;
                C* const pz = batch_at(A.fc, gc) + (ptrdiff_t)K * (ptrdiff_t)gc.ps;
                const auto c0 = leg_plane(pz + ((K & 1) ? 0 : (ptrdiff_t)gc.cs), on, cbytes);
                const auto c1 = leg_plane(pz + ((K & 1) ? (ptrdiff_t)gc.cs : 0), on, cbytes);
                leg_store(c0, coff0, (rsum * A.scale));
                leg_store(c1, coff1, (rsum * A.scale));
            }
            // both colours of plane a - NX
#pragma unroll
            for (int r = 0; r < 2; r++) {
                const bool od = r ? !par : par;  // the red point
                C* const rw = resl + pa1 * RESN + rwo[r];
                if (rw1[r]) rw[0] = od ? rr[r] : rbh[r];
                if (rw2[r]) rw[NCT - 1] = od ? rbh[r] : rr[r];
            }
        }
        // ---- shift
#pragma unroll
        for (int r = 0; r < 2; r++) {
            rbh[r] = sb[r];
            b0m[r] = b0c[r];
            b0c[r] = b0p[r];
#pragma unroll
            for (int i = 0; i < NX; i++) {
                x2[i][r] = x1[i][r];
                x1[i][r] = xn[i][r];
            }
#pragma unroll
            for (int i = NX - 1; i > 0; i--) fbh[i][r] = fbh[i - 1][r];
            fbh[0][r] = q.fb[r];
        }
        lds_barrier();
    };

    // first and last step: two more in front fill the start's planes
    const int as = (UP ? Z0 - (NX - 1 + NORM) : Z0 - NX) - (ZERO ? 0 : 2);
    const int ae = UP ? Z1 + NX - 1 + NORM : ZE + NX + 1;
    if constexpr (UP) {
        // the first step's coarse planes K and K + 1; the first step with an odd z stores a
        // plane, the one with an even z shifts (if it is the first: hand it plane K as the later one)
        const int K = (as + 1) >> 1;
        C e0[NE], e1[NE];
        load_e(K, e0);
        load_e(K + 1, e1);
        load_e(K + 2, epf[0]);
        load_e(K + 3, epf[1]);
        store_e(K, e0);
        store_e(K + 1, e1);
        __syncthreads();
        interp_e(K, v0c, v1c);
        interp_e(K + 1, v0n, v1n);
        if (kStepPar) {
#pragma unroll
            for (int r = 0; r < 2; r++) {
                v0n[r] = v0c[r];
                v1n[r] = v1c[r];
            }
        }
        __syncthreads();
    }
    using P0 = std::integral_constant<int, (S::H + kStepPar) & 1>;
    using P1 = std::integral_constant<int, (S::H + kStepPar + 1) & 1>;
    // steps between a load and its use: three, two where registers are short
    constexpr int LEAD = sizeof(C) == 8 && N == 2 ? 2 : 3;
    Feed q0, q1, q2, q3;
    load(P0{}, q0, as);
    load(P1{}, q1, as + 1);
    if constexpr (LEAD == 3) load(P0{}, q2, as + 2);
    const auto any_step = [&](auto par_tag, int a, const Feed& q, C (&ep)[NE]) {
        if (a - NX < 2 || a + 1 >= Nz) step(std::integral_constant<int, 2>{}, par_tag, a, q, ep);
        else if (edge) step(std::integral_constant<int, 1>{}, par_tag, a, q, ep);
        else step(std::integral_constant<int, 0>{}, par_tag, a, q, ep);
    };
    const auto next = [&](auto par_tag, Feed& two, Feed& three, int a) {
        if constexpr (LEAD == 3) load(std::integral_constant<int, 1 - decltype(par_tag)::value>{}, three, a + 3);
        else load(par_tag, two, a + 2);
    };
    for (int a = as; a <= ae; a += 4) {
        next(P0{}, q2, q3, a);
        any_step(P0{}, a, q0, epf[0]);
        if (a + 1 > ae) break;
        next(P1{}, q3, q0, a + 1);
        any_step(P1{}, a + 1, q1, epf[0]);
        if (a + 2 > ae) break;
        next(P0{}, q0, q1, a + 2);
        any_step(P0{}, a + 2, q2, epf[1]);
        if (a + 3 > ae) break;
        next(P1{}, q1, q2, a + 3);
        any_step(P1{}, a + 3, q3, epf[1]);
    }
    if constexpr (UP && NORM) block_max_to_w<S::NT / 64, false>(best, A.maxbits + blockIdx.y);
}

}  // namespace

// ------------------------------------------------------------------ launches
// Column of a workgroup per halo width: 512 threads, with FP64's registers all that a CU
// takes (in FP32 it takes two), each wavefront two rows of 32 compact points, so that
// a lane's x-neighbours are the lanes beside it.  The halo makes the work 1.3 to 1.7
// times the points (with 256 threads and two workgroups per CU in FP64 1.6 times for
// H = 3: 1.4 times as long).
template <int H>
struct LegPick;
template <> struct LegPick<2> { using S = LegShape<2, 58, 28>; };
template <> struct LegPick<3> { using S = LegShape<3, 58, 26>; };
template <> struct LegPick<4> { using S = LegShape<4, 54, 24>; };
template <> struct LegPick<5> { using S = LegShape<5, 54, 22>; };

// Planes per chunk: a chunk takes its planes and `extra` steps (filling the pipeline,
// the halo), the workgroups run in rounds of occ per CU.
static int leg_planes(long cols, int nz, int extra, int occ)
{
    long best = 0;
    int kz_best = 2;
    for (int nch = 1; nch <= (nz + 1) / 2; nch++) {
        const int kz = ((nz + nch - 1) / nch + 1) & ~1;
        const long wgs = cols * ((nz + kz - 1) / kz), cost = (wgs + 256 * occ - 1) / (256 * occ) * (kz + extra);
        if (nch == 1 || cost < best) {
            best = cost;
            kz_best = kz;
        }
        if (kz == 2) break;
    }
    return kz_best;
}

template <typename T, int N, int MODE, bool UP>
static void leg3(hipStream_t st, LegArgs<T> A)
{
    // a halo point per half sweep or residual that follows
    constexpr int H = UP ? 2 * N + (MODE != kLegRule && sizeof(T) == 8) : 2 * N + (MODE == kLegWarm);
    using S = typename LegPick<H>::S;
    A.nbx = ceil_div(A.g.nx - 2, S::TX);
    A.nby = ceil_div(A.g.ny - 2, S::TY);
    A.kz = leg_planes((long)A.nbx * A.nby * A.g.nb, A.g.nz - 2, 2 * H + 2 * N + 3, sizeof(T) == 8 ? 1 : 2);
    const dim3 grid((unsigned)((long)A.nbx * A.nby * ceil_div(A.g.nz - 2, A.kz)), A.g.nb);
    hipLaunchKernelGGL((k_leg3<T, N, MODE, UP, S>), grid, dim3(S::NT), 0, st, A);
}

template <typename T>
static LegArgs<T> leg_args(const LevelLeg& a, const T* u_in, const T* ring, const T* f, T* u_out, T* fc, const T* ec,
                           unsigned long long* maxbits)
{
    LegArgs<T> A{};
    A.u_in = u_in;
    A.ring = ring;
    A.f = f;
    A.u_out = u_out;
    A.fc = fc;
    A.ec = ec;
    A.g = a.g;
    A.gc = a.gc;
    A.h2 = (T)a.h2;
    A.inv2d = (T)(1.0 / 6.0);
    A.inv_h2 = (T)a.inv_h2;
    A.gr = grule<T>(a.rule);
    A.gcr = grule<T>(a.coarse_rule);
    A.rev = a.rev;
    A.maxbits = maxbits;
    return A;
}

template <int MODE, typename T>
static void stream_down(hipStream_t st, LegArgs<T> A, int n_pre, double out_scale)
{
    A.scale = (T)0.125 * (T)out_scale;
    if (n_pre == 1) leg3<T, 1, MODE, false>(st, A);
    else leg3<T, 2, MODE, false>(st, A);
}

template <typename T>
void launch_stream_down(hipStream_t st, const LevelLeg& a, int n_pre, const T* f, T* u, T* fc)
{
    stream_down<kLegRule>(st, leg_args<T>(a, u, u, f, u, fc, nullptr, nullptr), n_pre, 1.0);
}

template <typename T>
void launch_stream_up(hipStream_t st, const LevelLeg& a, int n_post, const T* u_in, const T* f, T* u_out, const T* ec)
{
    const LegArgs<T> A = leg_args<T>(a, u_in, u_in, f, u_out, nullptr, ec, nullptr);
    if (n_post == 1) leg3<T, 1, kLegRule, true>(st, A);
    else leg3<T, 2, kLegRule, true>(st, A);
}

void launch_stream0_down(hipStream_t st, const LevelLeg& a, int n_pre, const double* u_in, const double* f, double* u_out,
                         double* fc)
{
    stream_down<kLegWarm>(st, leg_args<double>(a, u_in, u_in, f, u_out, fc, nullptr, nullptr), n_pre, 1.0);
}

void launch_stream0_up(hipStream_t st, const LevelLeg& a, int n_post, const double* u_in, const double* ring,
                       const double* f, double* u_out, const double* ec, unsigned long long* maxbits)
{
    const LegArgs<double> A = leg_args<double>(a, u_in, ring, f, u_out, nullptr, ec, maxbits);
    if (n_post == 1) leg3<double, 1, kLegWarm, true>(st, A);
    else leg3<double, 2, kLegWarm, true>(st, A);
}

void launch_level0_down32(hipStream_t st, const LevelLeg& a, int n_pre, bool zero, const float* u_in, const float* f,
                          float* u_out, float* fc, double out_scale)
{
    const LegArgs<float> A = leg_args<float>(a, u_in, u_in, f, u_out, fc, nullptr, nullptr);
    if (zero) stream_down<kLegZero>(st, A, n_pre, out_scale);
    else stream_down<kLegWarm>(st, A, n_pre, out_scale);
}

void launch_level0_up32(hipStream_t st, const LevelLeg& a, const float* u_in, const float* ring, const float* f,
                        float* u_out, const float* ec)
{
    leg3<float, 1, kLegWarm, true>(st, leg_args<float>(a, u_in, ring, f, u_out, nullptr, ec, nullptr));
}

template void launch_stream_down<double>(hipStream_t, const LevelLeg&, int, const double*, double*, double*);
template void launch_stream_down<float>(hipStream_t, const LevelLeg&, int, const float*, float*, float*);
template void launch_stream_up<double>(hipStream_t, const LevelLeg&, int, const double*, const double*, double*, const double*);
template void launch_stream_up<float>(hipStream_t, const LevelLeg&, int, const float*, const float*, float*, const float*);

}  // namespace np
