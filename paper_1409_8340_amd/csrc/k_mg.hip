// k_mg.hip -- multigrid solver for the scalar potential on gfx950.
//
// The Poisson equation of Sec. 3.2, Delta_h mu = f (7-point stencil, plain
// wrap on periodic axes, Neumann reflection at open faces), is solved by
// V-cycles.  The smoother is the paper's pseudo-time relaxation: one
// Crank-Nicolson pseudo-step of d mu / d tau = Delta mu - f solved by a
// single Jacobi iteration is a damped Jacobi sweep,
//     mu <- mu + omega (f - A mu) / D,
// with omega = 2 h_tau S / (1 + h_tau S) set by the pseudo time step.
//
// Level operators are the finite-volume form of the stencil,
//     (A mu)_m = sum_a ap_a (mu_{m+a} - mu_m) + am_a (mu_{m-a} - mu_m),
// which is exactly Delta_h on the finest level (the boundary coefficient of
// an open face is twice the interior one, the Neumann ghost).  Periodic axes
// are coarsened by two; open axes keep nodes {0, 2, 4, ...} and the last node,
// so any node count coarsens, at the price of a non-uniform coarse spacing.
// Transfers are linear interpolation and its volume-weighted transpose.
//
// The restriction, the first residual and the mean map one thread to one
// (x, y) column of a 64 x 4 tile and march through a chunk of z planes.
#include "kernels.h"
#include "stencil.h"

#include <type_traits>

namespace tdgl {

struct MGCols {
    int lv, x, y, k0, k1;
    bool valid;
};

__device__ __forceinline__ MGCols mg_map(const MGLevel &L, int lb) {
    MGCols c;
    int t = lb;
    const int tx = t % L.tiles_x;
    t /= L.tiles_x;
    const int ty = t % L.tiles_y;
    const int tz = t / L.tiles_y;
    c.x = tx * MTX + (threadIdx.x & (MTX - 1));
    c.y = ty * MTY + (threadIdx.x / MTX);
    c.k0 = tz * L.chunk;
    c.k1 = min(c.k0 + L.chunk, L.nz);
    c.valid = (c.x < L.nx) && (c.y < L.ny);
    return c;
}

__device__ __forceinline__ int wrapi(int i, int n, int per) {
    if (i < 0) return per ? i + n : 0;
    if (i >= n) return per ? i - n : n - 1;
    return i;
}

// Poisson residual rows: the solve of this step ended at cycle c (or an
// earlier one) when row c is below max(mu_tol, mu_rtol * row 0).  Row c is
// written by the finest residual of cycle c.  Read by whole wavefronts
// (uniform control flow, full waves).
__device__ __forceinline__ float mg_threshold(const Inst &I) {
    return fmaxf(I.mu_tol, I.mu_rtol * row_max_wave(I.mures, I.rstride, 0));
}
__device__ __forceinline__ bool mg_done(const Inst &I, int c) {
    if (c >= I.mu_max_cycles) return true;
    // (row c in the lower half-wave, row 0 in the upper)
    const float m = row_max_half(I.mures, I.rstride, (threadIdx.x & 32) ? 0 : c);
    const float r = __shfl(m, 0, 64), r0 = __shfl(m, 32, 64);
    return r < fmaxf(I.mu_tol, I.mu_rtol * r0);
}

// Shared column context: coefficient values of the column and its x/y
// neighbour indices.
struct ColCoef {
    float apx, amx, apy, amy;
    int xm, xp, ym, yp;
};

__device__ __forceinline__ ColCoef col_coef(const MGLevel &L, int x, int y) {
    ColCoef c;
    c.apx = L.ap[0][x];
    c.amx = L.am[0][x];
    c.apy = L.ap[1][y];
    c.amy = L.am[1][y];
    c.xm = wrapi(x - 1, L.nx, L.per[0]);
    c.xp = wrapi(x + 1, L.nx, L.per[0]);
    c.ym = wrapi(y - 1, L.ny, L.per[1]);
    c.yp = wrapi(y + 1, L.ny, L.per[1]);
    return c;
}

// Residual r = rhs - A mu of the finest level before cycle cyc (the first, or
// any of a hierarchy of one level; k_mg_blk makes the others), evaluated in
// double precision from the stored single-precision iterate, and its max |r|
// into the cycle's convergence row.  Nothing when the previous cycle had
// already converged.
__global__ __launch_bounds__(256) void k_mg_residual(const Inst *__restrict__ insts,
                                                     const int *__restrict__ prefix, int ninst, int cyc) {
    __shared__ float red[4];
    const int ii = find_inst(prefix, ninst, blockIdx.x);
    const Inst &I = insts[ii];
    if (cyc > 0 && mg_done(I, cyc - 1)) return;
    const MGLevel &L = I.lev[0];
    const MGCols q = mg_map(L, blockIdx.x - prefix[ii]);
    float rmax = 0.f;
    if (q.valid) {
        const float *__restrict__ src = L.mu[0];
        const double fm = I.st->f_mean;
        const ColCoef c = col_coef(L, q.x, q.y);
        const long nxy = (long)L.nx * L.ny;
        const long col = (long)q.y * L.nx + q.x;
        const int zper = L.per[2];
        double mprev = src[wrapi(q.k0 - 1, L.nz, zper) * nxy + col];
        double mc = src[q.k0 * nxy + col];
        for (int k = q.k0; k < q.k1; ++k) {
            const double mnext = src[wrapi(k + 1, L.nz, zper) * nxy + col];
            const long pb = k * nxy;
            const double Amu =
                (double)c.apx * ((double)src[pb + q.y * (long)L.nx + c.xp] - mc) +
                (double)c.amx * ((double)src[pb + q.y * (long)L.nx + c.xm] - mc) +
                (double)c.apy * ((double)src[pb + c.yp * (long)L.nx + q.x] - mc) +
                (double)c.amy * ((double)src[pb + c.ym * (long)L.nx + q.x] - mc) +
                (double)L.ap[2][k] * (mnext - mc) + (double)L.am[2][k] * (mprev - mc);
            const double r = ((double)L.rhs[pb + col] - fm) - Amu;
            L.r[pb + col] = (float)r;
            const float ra = (float)fabs(r);
            rmax = (ra > rmax || ra != ra) ? ra : rmax;
            mprev = mc;
            mc = mnext;
        }
    }
    wg_max_to<256>(row_slot(I.mures, I.rstride, cyc, blockIdx.x), rmax, red);
}

// Restriction of the residual of level lv to the right side of level lv+1
// (volume-weighted transpose of linear interpolation, up to three fine
// indices per axis), followed by the first smoothing sweep of the coarse
// correction from a zero initial guess: e = omega rhs / D.
__global__ __launch_bounds__(256) void k_mg_restrict(const Inst *__restrict__ insts,
                                                     const int *__restrict__ prefix, int ninst,
                                                     int lv, int cyc, float omega) {
    const int ii = find_inst(prefix, ninst, blockIdx.x);
    const Inst &I = insts[ii];
    if (mg_done(I, cyc)) return;
    const MGLevel &F = I.lev[lv];
    const MGLevel &C = I.lev[lv + 1];
    const MGCols q = mg_map(C, blockIdx.x - prefix[ii]);
    if (!q.valid) return;
    int fx[3], fy[3];
    float wx[3], wy[3];
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        fx[a] = F.rk[0][3 * q.x + a];
        wx[a] = F.rw[0][3 * q.x + a];
        fy[a] = F.rk[1][3 * q.y + a];
        wy[a] = F.rw[1][3 * q.y + a];
    }
    const float Dxy = C.ap[0][q.x] + C.am[0][q.x] + C.ap[1][q.y] + C.am[1][q.y];
    const long fnxy = (long)F.nx * F.ny;
    const long cnxy = (long)C.nx * C.ny;
    for (int K = q.k0; K < q.k1; ++K) {
        float s = 0.f;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            const float wz = F.rw[2][3 * K + c];
            const long pb = (long)F.rk[2][3 * K + c] * fnxy;
#pragma unroll
            for (int b2 = 0; b2 < 3; ++b2) {
                const long rb = pb + (long)fy[b2] * F.nx;
                const float wzy = wz * wy[b2];
#pragma unroll
                for (int a = 0; a < 3; ++a) s += wzy * wx[a] * F.r[rb + fx[a]];
            }
        }
        const long m = K * cnxy + (long)q.y * C.nx + q.x;
        C.rhs[m] = s;
        const float D = -(Dxy + C.ap[2][K] + C.am[2][K]);
        C.mu[0][m] = (D != 0.f) ? omega * s / D : 0.f;
    }
}

// Coarse-to-fine correction mu += P e_c of the finest level (linear
// interpolation per axis).
__global__ __launch_bounds__(256) void k_mg_prolong(const Inst *__restrict__ insts,
                                                    const int *__restrict__ prefix, int ninst,
                                                    int cyc) {
    const int ii = find_inst(prefix, ninst, blockIdx.x);
    const Inst &I = insts[ii];
    if (mg_done(I, cyc)) return;
    const MGLevel &F = I.lev[0];
    const MGLevel &C = I.lev[1];
    const MGCols q = mg_map(F, blockIdx.x - prefix[ii]);
    if (!q.valid) return;
    const int kx0 = F.pk[0][2 * q.x], kx1 = F.pk[0][2 * q.x + 1];
    const float wx0 = F.pw[0][2 * q.x], wx1 = F.pw[0][2 * q.x + 1];
    const int ky0 = F.pk[1][2 * q.y], ky1 = F.pk[1][2 * q.y + 1];
    const float wy0 = F.pw[1][2 * q.y], wy1 = F.pw[1][2 * q.y + 1];
    const float *__restrict__ ec = C.mu[0];
    float *__restrict__ mf = F.mu[0];
    const long cnxy = (long)C.nx * C.ny, fnxy = (long)F.nx * F.ny;
    for (int k = q.k0; k < q.k1; ++k) {
        const int kz0 = F.pk[2][2 * k], kz1 = F.pk[2][2 * k + 1];
        const float wz0 = F.pw[2][2 * k], wz1 = F.pw[2][2 * k + 1];
        const long b0 = kz0 * cnxy, b1 = kz1 * cnxy;
        const float e =
            wz0 * (wy0 * (wx0 * ec[b0 + (long)ky0 * C.nx + kx0] + wx1 * ec[b0 + (long)ky0 * C.nx + kx1]) +
                   wy1 * (wx0 * ec[b0 + (long)ky1 * C.nx + kx0] + wx1 * ec[b0 + (long)ky1 * C.nx + kx1])) +
            wz1 * (wy0 * (wx0 * ec[b1 + (long)ky0 * C.nx + kx0] + wx1 * ec[b1 + (long)ky0 * C.nx + kx1]) +
                   wy1 * (wx0 * ec[b1 + (long)ky1 * C.nx + kx0] + wx1 * ec[b1 + (long)ky1 * C.nx + kx1]));
        mf[k * fnxy + (long)q.y * F.nx + q.x] += e;
    }
}

// Smoothing passes of level lv on MGB_X x MGB_Y x MGB_Z blocks, from mu[isrc]
// into the other buffer: the correction of the next coarser level first (PRO,
// mu += P e_c by linear interpolation per axis), then S damped Jacobi sweeps
//   mu <- mu + omega (rhs - A mu) / D,
// then the residual r = rhs - A mu in double precision from the
// single-precision iterate (RES; on level 0 with its max |r| into the next
// cycle's convergence row).  Level 0 subtracts the weighted mean of f from its
// right side (projection onto the range of the singular operator).
// A pass over a coarse level is a chain of memory latencies of 5 us and more,
// whatever its size, and each level above the tail had five of them, the
// finest six.  A thread holds one (x, y) column of the block with a halo of one
// node per sweep (and one for the residual), its planes in registers, the
// block's planes in LDS; what a sweep gets wrong at the halo's rim moves in by
// one node per sweep and never reaches the block.  The convergence rows are
// read behind the block's loads, and the work-groups of a cycle that has ended
// stop there: they took 5 to 7 us a launch to compute what was not stored
// (replayed steps of 256 x 101 x 33, which launch every cycle, 1944 -> 1606 us).
// The operations on a node and their order are those of one sweep, correction
// or residual at a time, so are the bits.
// Below 192 x 101 x 33: correction and two sweeps of 96 x 51 x 17 and 48 x 26 x
// 9 nodes 10 us each (15 as three launches), a sweep and the residual 6.5 (10);
// of the finest level two sweeps 11 us (16), two and the residual 19 (25).  The
// finest level's correction stays a pass of its own (6 us): with the halo's
// interpolation in front, its two sweeps took 27 us.  A run 9.9 -> 9.5 ms.
template <bool PRO, int S, bool RES>
__global__ __launch_bounds__(mgb_threads(S + RES)) void k_mg_blk(const Inst *__restrict__ insts,
                                                                 const int *__restrict__ prefix, int ninst, int lv,
                                                                 int isrc, int cyc, float omega) {
    constexpr int H = S + RES, W = MGB_X + 2 * H, HT = MGB_Y + 2 * H, NP = MGB_Z + 2 * H, NT = mgb_threads(H);
    __shared__ float buf[2][NP][W * HT];
    __shared__ float red[NT / 64];
    const int ii = find_inst(prefix, ninst, blockIdx.x);
    const Inst &I = insts[ii];
    const MGLevel &L = I.lev[lv];
    const int nx = L.nx, ny = L.ny, nz = L.nz, nxy = nx * ny;
    int b = blockIdx.x - prefix[ii];
    const int bx = (nx + MGB_X - 1) / MGB_X, by = (ny + MGB_Y - 1) / MGB_Y;
    const int x0 = b % bx * MGB_X;
    b /= bx;
    const int y0 = b % by * MGB_Y, k0 = b / by * MGB_Z;
    const int t = min((int)threadIdx.x, W * HT - 1);  // (the last threads repeat the last column)
    const int tx = t % W, ty = t / W, gx = x0 - H + tx, gy = y0 - H + ty;
    // the slot's node: an image on a periodic axis; slots outside an open one
    // are not read (they hold some node of the grid)
    auto image = [](int g, int n, int per) { return per ? ((g % n) + n) % n : min(max(g, 0), n - 1); };
    const int x = image(gx, nx, L.per[0]), y = image(gy, ny, L.per[1]);
    const bool in = (int)threadIdx.x < W * HT && tx >= H && tx < H + MGB_X && ty >= H && ty < H + MGB_Y && gx < nx && gy < ny;
    // neighbour slots (the node itself beyond an open face, as wrapi() has it,
    // and at the halo's rim)
    const int sxm = (tx == 0 || (!L.per[0] && gx == 0)) ? t : t - 1;
    const int sxp = (tx == W - 1 || (!L.per[0] && gx == nx - 1)) ? t : t + 1;
    const int sym = (ty == 0 || (!L.per[1] && gy == 0)) ? t : t - W;
    const int syp = (ty == HT - 1 || (!L.per[1] && gy == ny - 1)) ? t : t + W;
    const float *__restrict__ src = L.mu[isrc];
    float *__restrict__ dst = L.mu[isrc ^ 1];
    const float *__restrict__ rhsp = L.rhs;
    const float apx = L.ap[0][x], amx = L.am[0][x], apy = L.ap[1][y], amy = L.am[1][y];
    const double fmd = lv == 0 ? I.st->f_mean : 0.0;
    const float fm = (float)fmd;
    const int col = y * nx + x;
    float v[NP], rh[NP], apz[NP], amz[NP];
#pragma unroll
    for (int q = 0; q < NP; ++q) {
        const int k = image(k0 - H + q, nz, L.per[2]);
        v[q] = src[k * nxy + col];
        rh[q] = rhsp[k * nxy + col];
        apz[q] = scalar_f(L.ap[2][k]);
        amz[q] = scalar_f(L.am[2][k]);
    }
    if (PRO) {
        const MGLevel &C = I.lev[lv + 1];
        const float *__restrict__ ec = C.mu[0];
        const int cnx = C.nx, cnxy = C.nx * C.ny;
        const int kx0 = L.pk[0][2 * x], kx1 = L.pk[0][2 * x + 1];
        const float wx0 = L.pw[0][2 * x], wx1 = L.pw[0][2 * x + 1];
        const int ky0 = L.pk[1][2 * y], ky1 = L.pk[1][2 * y + 1];
        const float wy0 = L.pw[1][2 * y], wy1 = L.pw[1][2 * y + 1];
        const int c00 = ky0 * cnx + kx0, c01 = ky0 * cnx + kx1, c10 = ky1 * cnx + kx0, c11 = ky1 * cnx + kx1;
#pragma unroll
        for (int q = 0; q < NP; ++q) {
            const int k = image(k0 - H + q, nz, L.per[2]);
            const float wz0 = scalar_f(L.pw[2][2 * k]), wz1 = scalar_f(L.pw[2][2 * k + 1]);
            const int b0 = __builtin_amdgcn_readfirstlane(L.pk[2][2 * k]) * cnxy;
            const int b1 = __builtin_amdgcn_readfirstlane(L.pk[2][2 * k + 1]) * cnxy;
            const float e = wz0 * (wy0 * (wx0 * ec[b0 + c00] + wx1 * ec[b0 + c01]) +
                                   wy1 * (wx0 * ec[b0 + c10] + wx1 * ec[b0 + c11])) +
                            wz1 * (wy0 * (wx0 * ec[b1 + c00] + wx1 * ec[b1 + c01]) +
                                   wy1 * (wx0 * ec[b1 + c10] + wx1 * ec[b1 + c11]));
            v[q] += e;
        }
    }
    if (__ballot(mg_done(I, cyc)) != 0) return;  // (one answer for all)
#pragma unroll
    for (int q = 0; q < NP; ++q) buf[0][q][t] = v[q];
    // z neighbours of plane q: the plane itself beyond an open face
    auto zlo = [&](int q) { return !L.per[2] && k0 - H + q == 0 ? v[q] : v[q - 1]; };
    auto zhi = [&](int q) { return !L.per[2] && k0 - H + q == nz - 1 ? v[q] : v[q + 1]; };
#pragma unroll
    for (int s = 0; s < S; ++s) {
        __syncthreads();
        float nv[NP];
        // (planes that the block's own do not depend on any more are left out)
#pragma unroll
        for (int q = s + 1; q < NP - 1 - s; ++q) {
            const float *P = buf[s & 1][q];
            const float mc = v[q], mnext = zhi(q), mprev = zlo(q);
            const float Amu = apx * (P[sxp] - mc) + amx * (P[sxm] - mc) + apy * (P[syp] - mc) + amy * (P[sym] - mc) +
                              apz[q] * (mnext - mc) + amz[q] * (mprev - mc);
            const float D = -(apx + amx + apy + amy + apz[q] + amz[q]);
            const float rhs = rh[q] - fm;
            nv[q] = (D != 0.f) ? mc + omega * (rhs - Amu) / D : mc;
        }
#pragma unroll
        for (int q = s + 1; q < NP - 1 - s; ++q) {
            v[q] = nv[q];
            if (s + 1 < S || RES) buf[(s & 1) ^ 1][q][t] = nv[q];
        }
    }
    const int k1 = min(MGB_Z, nz - k0);
    if (in) {
#pragma unroll
        for (int q = 0; q < MGB_Z; ++q)
            if (q < k1) dst[(k0 + q) * nxy + col] = v[H + q];
    }
    if (RES) {
        float rmax = 0.f;
        __syncthreads();
#pragma unroll
        for (int c = 0; c < MGB_Z; ++c) {
            const int q = H + c;
            const float *P = buf[S & 1][q];
            const double mc = v[q], mnext = zhi(q), mprev = zlo(q);
            const double Amu = (double)apx * ((double)P[sxp] - mc) + (double)amx * ((double)P[sxm] - mc) +
                               (double)apy * ((double)P[syp] - mc) + (double)amy * ((double)P[sym] - mc) +
                               (double)apz[q] * (mnext - mc) + (double)amz[q] * (mprev - mc);
            const double r = ((double)rh[q] - fmd) - Amu;
            if (in && c < k1) {
                L.r[(k0 + c) * nxy + col] = (float)r;
                const float ra = (float)fabs(r);
                rmax = (ra > rmax || ra != ra) ? ra : rmax;
            }
        }
        if (lv == 0 && cyc + 1 < I.mu_max_cycles)
            wg_max_to<NT>(row_slot(I.mures, I.rstride, cyc + 1, blockIdx.x), rmax, red);
    }
}
#define TDGL_MG_INST(P, S, R) \
    template __global__ void k_mg_blk<P, S, R>(const Inst *, const int *, int, int, int, int, float);
TDGL_MG_INST(false, 1, true)
TDGL_MG_INST(true, 2, false)
TDGL_MG_INST(false, 2, false)
TDGL_MG_INST(false, 2, true)
#undef TDGL_MG_INST

// Coarsest level L of a work-group: Jacobi sweeps in double precision on an
// FP32 iterate until the residual falls below 1e-6 of the right side or 4000
// sweeps, after projecting the right side rhs - fm onto the range (zero
// volume-weighted mean).  Starts from mu0, or from zero without one; returns
// the LDS buffer with the result and the mean to subtract.
// A thread keeps its nodes' coefficients and right sides in registers, and a
// sweep ends at one barrier with a vote on the residual, since only whether
// the maximum exceeds the threshold matters.  A sweep is a chain of some 20
// FP64 operations between two LDS round trips, so everything else is kept out
// of it: the vote of a sweep is read with the next sweep's loads (that sweep
// is dropped before it stores when the vote has closed the iteration), buffers
// and words have fixed addresses over six unrolled sweeps, and threads without
// a node sweep a slot of their own under an infinite threshold.  Through global memory, with the maximum reduced
// every sweep over 1024 threads, a solve took 465 us on average on the 12 x 8
// x 3 nodes below 192 x 101 x 33, three quarters of that box's step, and 87 us
// with the vote read behind its own barrier and addresses made per sweep.  The values are those of that
// form, bit for bit: the quotient by D is its reciprocal's product corrected
// once with the exact remainder, which rounds as the division does (Markstein,
// IBM J. Res. Dev. 34, 1990).  (A direct solve through the axes' modes takes
// 7 us, but what it takes away from the stop rule's error reaches the ninth
// digit of K.)
// NPT: nodes per thread (1 where N fits the work-group, else 4).
template <int NPT>
__device__ __forceinline__ const float *mg_coarsest(const MGLevel &L, const float *rhs, double fm, const float *mu0,
                                                    float &mmean) {
    constexpr int CAP = NPT * CO_THREADS;
    __shared__ float cb[2][CAP];
    __shared__ double red[CO_THREADS / 64];
    __shared__ double sh_v;
    __shared__ int open[3];
    const int N = L.N, nt = (int)blockDim.x, nw = nt >> 6;
    auto sum = [&](double v) {
        for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
        __syncthreads();
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
        __syncthreads();
        double s = 0.0;
        for (int i = 0; i < nw; ++i) s += red[i];
        return s;
    };
    int at[NPT][7];                      // the node and its six neighbours
    double co[NPT][6], D[NPT], rD[NPT], V[NPT], d0[NPT];
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
        const int m = (int)threadIdx.x + i * nt, mm = m < N ? m : 0;
        const int x = mm % L.nx, y = (mm / L.nx) % L.ny, z = mm / (L.nx * L.ny);
        const int xm = wrapi(x - 1, L.nx, L.per[0]), xp = wrapi(x + 1, L.nx, L.per[0]);
        const int ym = wrapi(y - 1, L.ny, L.per[1]), yp = wrapi(y + 1, L.ny, L.per[1]);
        const int zm = wrapi(z - 1, L.nz, L.per[2]), zp = wrapi(z + 1, L.nz, L.per[2]);
        const int nx = L.nx, nxy = L.nx * L.ny;
        at[i][0] = z * nxy + y * nx + xp;
        at[i][1] = z * nxy + y * nx + xm;
        at[i][2] = z * nxy + yp * nx + x;
        at[i][3] = z * nxy + ym * nx + x;
        at[i][4] = zp * nxy + y * nx + x;
        at[i][5] = zm * nxy + y * nx + x;
        at[i][6] = m;
        cb[0][m] = mu0 && m < N ? mu0[m] : 0.f;
        co[i][0] = (double)L.ap[0][x];
        co[i][1] = (double)L.am[0][x];
        co[i][2] = (double)L.ap[1][y];
        co[i][3] = (double)L.am[1][y];
        co[i][4] = (double)L.ap[2][z];
        co[i][5] = (double)L.am[2][z];
        D[i] = -((double)L.ap[0][x] + L.am[0][x] + L.ap[1][y] + L.am[1][y] + L.ap[2][z] + L.am[2][z]);
        rD[i] = D[i] != 0.0 ? 1.0 / D[i] : 0.0;  // 0: the node keeps its value
        V[i] = (double)L.vol[0][x] * L.vol[1][y] * L.vol[2][z];
        d0[i] = (double)rhs[mm] - fm;
        // volume-weighted mean of the right side
        if (m < N) s += V[i] * d0[i];
    }
    if (threadIdx.x < 3) open[threadIdx.x] = 0;
    s = sum(s);
    const double rmean = s / L.vsum;
    double rnorm = 0.0;
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
        d0[i] -= rmean;
        if ((int)threadIdx.x + i * nt < N) rnorm = fmax(rnorm, fabs(d0[i]));
    }
    for (int o = 32; o > 0; o >>= 1) rnorm = fmax(rnorm, __shfl_xor(rnorm, o, 64));
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = rnorm;
    __syncthreads();
    if (threadIdx.x == 0) {
        double mx = 0.0;
        for (int i = 0; i < nw; ++i) mx = fmax(mx, red[i]);
        sh_v = mx;
    }
    __syncthreads();
    double thr[NPT];
#pragma unroll
    for (int i = 0; i < NPT; ++i)
        thr[i] = (int)threadIdx.x + i * nt < N ? 1e-6 * sh_v : (double)INFINITY;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const bool busy = w * 64 < N;  // some node of the wavefront's is one of the level's
    // sweep it = J mod 6 from cb[J & 1]; false: the sweep before ended the
    // iteration (its result is in cb[J & 1])
    auto sweep = [&](auto jc, int it) __attribute__((always_inline)) {
        constexpr int J = decltype(jc)::value, ph = J % 3, pq = (ph + 2) % 3, pn = (ph + 1) % 3;
        const float *a = cb[J & 1];
        float *bq = cb[(J & 1) ^ 1];
        const int going = open[pq];  // the vote of the sweep before
        float nv[NPT];
        bool over = false;
        if (busy) {
#pragma unroll
            for (int i = 0; i < NPT; ++i) {
                const double mc = a[at[i][6]];
                const double Amu = co[i][0] * (a[at[i][0]] - mc) + co[i][1] * (a[at[i][1]] - mc) +
                                   co[i][2] * (a[at[i][2]] - mc) + co[i][3] * (a[at[i][3]] - mc) +
                                   co[i][4] * (a[at[i][4]] - mc) + co[i][5] * (a[at[i][5]] - mc);
                const double r = d0[i] - Amu;
                const double x = 0.9 * r, q = x * rD[i];
                const double quo = __builtin_fma(__builtin_fma(-q, D[i], x), rD[i], q);
                over = over || fabs(r) > thr[i];
                nv[i] = (rD[i] != 0.0) ? (float)(mc + quo) : (float)mc;
            }
        }
        if (it > 0 && !__builtin_amdgcn_readfirstlane(going)) return false;
        if (busy) {
#pragma unroll
            for (int i = 0; i < NPT; ++i) bq[at[i][6]] = nv[i];
            if (__ballot(over) != 0) open[ph] = 1;
        }
        // the next sweep's word: read last in the sweep before this one
        if (w == 0) open[pn] = 0;
        __syncthreads();
        return true;
    };
    int ph = 0;  // the buffer with the result
    for (int it = 0; it < 4000; ++it) {
        ph = 0;
        if (!sweep(std::integral_constant<int, 0>{}, it)) break;
        ph = 1;
        if (++it >= 4000 || !sweep(std::integral_constant<int, 1>{}, it)) break;
        ph = 0;
        if (++it >= 4000 || !sweep(std::integral_constant<int, 2>{}, it)) break;
        ph = 1;
        if (++it >= 4000 || !sweep(std::integral_constant<int, 3>{}, it)) break;
        ph = 0;
        if (++it >= 4000 || !sweep(std::integral_constant<int, 4>{}, it)) break;
        ph = 1;
        if (++it >= 4000 || !sweep(std::integral_constant<int, 5>{}, it)) break;
        ph = 0;
    }
    float *a = cb[ph];
    // shift to zero weighted mean
    double sm = 0.0;
#pragma unroll
    for (int i = 0; i < NPT; ++i)
        if ((int)threadIdx.x + i * nt < N) sm += V[i] * a[at[i][6]];
    sm = sum(sm);
    mmean = (float)(sm / L.vsum);
    return a;
}

// The coarse end of a V-cycle in one work-group per instance: levels
// I.mg_tail and coarser, from the restriction of the next finer level's
// residual to the correction of level I.mg_tail, with the iterates and right
// sides in LDS (the residual takes the place of the level's first iterate,
// which the smoothing has used up).  The operations and their order are those
// of the per-level kernels, so are the bits.  A launch of these levels' kernels
// takes 5 to 7 us, whatever its size; here an operation takes one barrier.
// The levels' tables come to LDS in one piece, since a chain of pointer, table
// and value loads costs an operation as much as a launch does.
// (TL false, for an instance whose coarsest level's table is larger than LDS:
// read where it is.)  A hierarchy of one level (tiny grids) is solved directly: its right side is
// f minus its weighted mean and the iterate starts from the stored mu.
// 192 x 101 x 33 nodes (tail 24 x 14 x 5 and 12 x 8 x 3), per V-cycle: 78 us,
// nearly all of it the coarsest level's sweeps, for seven launches of 125 us;
// a run of six steps 11.6 -> 10.2 ms.
template <int NPT, bool TL>
__global__ __launch_bounds__(CO_THREADS) void k_mg_tail(const Inst *__restrict__ insts, int ninst, int cyc,
                                                        float omega) {
    extern __shared__ float tail_sm[];
    const Inst &I = insts[blockIdx.x];
    if (!I.driven || I.fft || TL != (I.mg_tlds != 0) || mg_done(I, cyc)) return;
    const int last = I.nlev - 1, lt = I.mg_tail, nt = (int)blockDim.x;
    // the levels' sizes and tables, from level lt - 1 on (see MgTab), then 3 N
    // floats per level: its iterates and right side
    const int *tab = TL ? (const int *)tail_sm : I.mg_tab;
    if (TL)
        for (int i = threadIdx.x; i < I.mg_words; i += nt) ((int *)tail_sm)[i] = I.mg_tab[i];
    const float *ftab = (const float *)tab;
    auto lev = [&](int l) {
        MgTab v;
        const int *h = tab + (l - lt + 1) * MG_TAB_HEAD;
        int w[MG_TAB_HEAD];
#pragma unroll
        for (int i = 0; i < MG_TAB_HEAD; ++i) w[i] = __builtin_amdgcn_readfirstlane(h[i]);
        v.nx = w[0]; v.ny = w[1]; v.nz = w[2]; v.N = w[3];
        v.px = w[4]; v.py = w[5]; v.pz = w[6];
        v.coef = w[7]; v.pro = w[8]; v.res = w[9];
        return v;
    };
    auto restrict_to = [&](const MgTab &F, const MgTab &C, const float *r, float *rhs, float *mu0) {
        const int Sc = C.nx + C.ny + C.nz, fnx = F.nx, fnxy = F.nx * F.ny;
        for (int m = threadIdx.x; m < C.N; m += nt) {
            const int x = m % C.nx, yk = m / C.nx, y = yk % C.ny, K = yk / C.ny;
            const int o[3] = {F.res + 3 * x, F.res + 3 * (C.nx + y), F.res + 3 * (C.nx + C.ny + K)};
            int f[3][3];
            float w[3][3];
#pragma unroll
            for (int ax = 0; ax < 3; ++ax)
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    f[ax][q] = tab[o[ax] + q];
                    w[ax][q] = ftab[o[ax] + 3 * Sc + q];
                }
            float v[27];
#pragma unroll
            for (int q = 0; q < 27; ++q) v[q] = r[f[2][q / 9] * fnxy + f[1][q / 3 % 3] * fnx + f[0][q % 3]];
            float s = 0.f;
#pragma unroll
            for (int q = 0; q < 27; ++q) {
                const float wzy = w[2][q / 9] * w[1][q / 3 % 3];
                s += wzy * w[0][q % 3] * v[q];
            }
            rhs[m] = s;
            const float *ap = ftab + C.coef, *am = ap + Sc;
            const float Dxy = ap[x] + am[x] + ap[C.nx + y] + am[C.nx + y];
            const float D = -(Dxy + ap[C.nx + C.ny + K] + am[C.nx + C.ny + K]);
            mu0[m] = (D != 0.f) ? omega * s / D : 0.f;
        }
    };
    // node m of a level: its coefficients and neighbours
    struct Node {
        float apx, amx, apy, amy, apz, amz;
        int xm, xp, ym, yp, zm, zp;
    };
    auto node = [&](const MgTab &L, int m) {
        Node c;
        const int nx = L.nx, nxy = L.nx * L.ny, S = L.nx + L.ny + L.nz;
        const int x = m % nx, yk = m / nx, y = yk % L.ny, k = yk / L.ny;
        const float *ap = ftab + L.coef, *am = ap + S;
        c.apx = ap[x];
        c.amx = am[x];
        c.apy = ap[nx + y];
        c.amy = am[nx + y];
        c.apz = ap[nx + L.ny + k];
        c.amz = am[nx + L.ny + k];
        c.xm = m - x + wrapi(x - 1, nx, L.px);
        c.xp = m - x + wrapi(x + 1, nx, L.px);
        c.ym = m + (wrapi(y - 1, L.ny, L.py) - y) * nx;
        c.yp = m + (wrapi(y + 1, L.ny, L.py) - y) * nx;
        c.zm = m + (wrapi(k - 1, L.nz, L.pz) - k) * nxy;
        c.zp = m + (wrapi(k + 1, L.nz, L.pz) - k) * nxy;
        return c;
    };
    auto smooth = [&](const MgTab &L, const float *src, float *dst, const float *rhsp) {
        for (int m = threadIdx.x; m < L.N; m += nt) {
            const Node c = node(L, m);
            const float mc = src[m];
            const float Amu = c.apx * (src[c.xp] - mc) + c.amx * (src[c.xm] - mc) + c.apy * (src[c.yp] - mc) +
                              c.amy * (src[c.ym] - mc) + c.apz * (src[c.zp] - mc) + c.amz * (src[c.zm] - mc);
            const float D = -(c.apx + c.amx + c.apy + c.amy + c.apz + c.amz);
            const float rhs = rhsp[m];
            dst[m] = (D != 0.f) ? mc + omega * (rhs - Amu) / D : mc;
        }
    };
    auto residual = [&](const MgTab &L, const float *src, float *r, const float *rhsp) {
        for (int m = threadIdx.x; m < L.N; m += nt) {
            const Node c = node(L, m);
            const double mc = src[m];
            const double Amu = (double)c.apx * ((double)src[c.xp] - mc) + (double)c.amx * ((double)src[c.xm] - mc) +
                               (double)c.apy * ((double)src[c.yp] - mc) + (double)c.amy * ((double)src[c.ym] - mc) +
                               (double)c.apz * ((double)src[c.zp] - mc) + (double)c.amz * ((double)src[c.zm] - mc);
            r[m] = (float)((double)rhsp[m] - Amu);
        }
    };
    auto prolong = [&](const MgTab &F, const MgTab &C, const float *ec, float *mf) {
        const int cnx = C.nx, cnxy = C.nx * C.ny, nx = F.nx, S2 = 2 * (F.nx + F.ny + F.nz);
        for (int m = threadIdx.x; m < F.N; m += nt) {
            const int x = m % nx, yk = m / nx, y = yk % F.ny, k = yk / F.ny;
            const int ox = F.pro + 2 * x, oy = F.pro + 2 * (nx + y), oz = F.pro + 2 * (nx + F.ny + k);
            const int kx0 = tab[ox], kx1 = tab[ox + 1], ky0 = tab[oy], ky1 = tab[oy + 1];
            const float wx0 = ftab[ox + S2], wx1 = ftab[ox + S2 + 1];
            const float wy0 = ftab[oy + S2], wy1 = ftab[oy + S2 + 1];
            const float wz0 = ftab[oz + S2], wz1 = ftab[oz + S2 + 1];
            const int b0 = tab[oz] * cnxy, b1 = tab[oz + 1] * cnxy;
            const float e = wz0 * (wy0 * (wx0 * ec[b0 + ky0 * cnx + kx0] + wx1 * ec[b0 + ky0 * cnx + kx1]) +
                                   wy1 * (wx0 * ec[b0 + ky1 * cnx + kx0] + wx1 * ec[b0 + ky1 * cnx + kx1])) +
                            wz1 * (wy0 * (wx0 * ec[b1 + ky0 * cnx + kx0] + wx1 * ec[b1 + ky0 * cnx + kx1]) +
                                   wy1 * (wx0 * ec[b1 + ky1 * cnx + kx0] + wx1 * ec[b1 + ky1 * cnx + kx1]));
            mf[m] += e;
        }
    };

    const MGLevel &T = I.lev[last];
    float mmean;
    if (last == 0) {
        const float *a = mg_coarsest<NPT>(T, T.rhs, I.st->f_mean, T.mu[0], mmean);
        for (int m = threadIdx.x; m < T.N; m += nt) T.mu[0][m] = a[m] - mmean;
        return;
    }
    // down
    __syncthreads();
    float *base = tail_sm + (TL ? I.mg_words : 0);
    {
        const MgTab C = lev(lt);
        restrict_to(lev(lt - 1), C, I.lev[lt - 1].r, base + 2 * C.N, base);
    }
    __syncthreads();
    for (int l = lt; l < last; ++l) {
        const MgTab L = lev(l), C = lev(l + 1);
        float *m0 = base, *m1 = base + L.N, *rh = base + 2 * L.N, *next = base + 3 * L.N;
        smooth(L, m0, m1, rh);
        __syncthreads();
        residual(L, m1, m0, rh);
        __syncthreads();
        restrict_to(L, C, m0, next + 2 * C.N, next);
        __syncthreads();
        base = next;
    }
    // coarsest
    const float *a = mg_coarsest<NPT>(T, base + 2 * T.N, 0.0, nullptr, mmean);
    if (lt == last) {
        for (int m = threadIdx.x; m < T.N; m += nt) T.mu[0][m] = a[m] - mmean;
        return;
    }
    float *e = base;
    for (int m = threadIdx.x; m < T.N; m += nt) e[m] = a[m] - mmean;
    __syncthreads();
    // up
    for (int l = last - 1; l >= lt; --l) {
        const MgTab L = lev(l);
        base -= 3 * L.N;
        float *m0 = base, *m1 = base + L.N, *rh = base + 2 * L.N;
        prolong(L, lev(l + 1), e, m1);
        __syncthreads();
        smooth(L, m1, m0, rh);
        __syncthreads();
        smooth(L, m0, m1, rh);
        __syncthreads();
        e = m1;
    }
    const MGLevel &L = I.lev[lt];
    for (int m = threadIdx.x; m < L.N; m += nt) L.mu[0][m] = e[m];
}
template __global__ void k_mg_tail<1, true>(const Inst *, int, int, float);
template __global__ void k_mg_tail<4, true>(const Inst *, int, int, float);
template __global__ void k_mg_tail<1, false>(const Inst *, int, int, float);
template __global__ void k_mg_tail<4, false>(const Inst *, int, int, float);

// End of a Poisson solve: number of cycles and final residual; clears the
// cycle words.  One thread per instance.
__global__ __launch_bounds__(FIN_THREADS) void k_mg_finalize(const Inst *__restrict__ insts, int ninst,
                                                               int count_step) {
    // one work-group per instance: the first wavefront scans the rows, then
    // all threads clear them
    const int ii = blockIdx.x;
    if (ii >= ninst) return;
    const Inst &I = insts[ii];
    if (!I.driven || I.fft) return;
    DevState *st = I.st;
    if (threadIdx.x < 64) {
        int cycles = I.mu_max_cycles, capped = 1;
        const float thr = mg_threshold(I);
        float last = row_max_wave(I.mures, I.rstride, I.mu_max_cycles - 1);
        for (int c = 0; c < I.mu_max_cycles; ++c) {
            const float r = row_max_wave(I.mures, I.rstride, c);
            if (r < thr) { cycles = c; capped = 0; last = r; break; }
        }
        if (threadIdx.x == 0) {
            st->mu_cycles = cycles;
            st->mu_capped = capped;
            st->mu_last_res = last;
            if (count_step) {
                st->acc_mu_cycles += cycles;
                st->acc_mu_capped += capped;
            }
        }
    }
    __syncthreads();
    const int words = I.mu_max_cycles * NSLOT;
    for (int w = threadIdx.x; w < words; w += FIN_THREADS) I.mures[(size_t)w * I.rstride] = 0u;
}

// Partial sums of V mu (which = 0) or V f (which = 1) on level 0 for the
// weighted mean.
__global__ __launch_bounds__(256) void k_mu_mean_partial(const Inst *__restrict__ insts,
                                                         const int *__restrict__ prefix, int ninst,
                                                         int which) {
    __shared__ double red[4];
    const int ii = find_inst(prefix, ninst, blockIdx.x);
    const Inst &I = insts[ii];
    const MGLevel &L = I.lev[0];
    const int lb = blockIdx.x - prefix[ii];
    const MGCols q = mg_map(L, lb);
    double acc = 0.0;
    if (q.valid) {
        const double vxy = (double)L.vol[0][q.x] * L.vol[1][q.y];
        const long nxy = (long)L.nx * L.ny, col = (long)q.y * L.nx + q.x;
        const gf1 *src = (const gf1 *)(which ? L.rhs : L.mu[0]);
        const gf1 *volz = (const gf1 *)L.vol[2];
        // eight planes' loads in flight before they are summed in plane order
        constexpr int KB = 8;
        int k = q.k0;
        for (; k + KB <= q.k1; k += KB) {
            float v[KB], wv[KB];
#pragma unroll
            for (int c = 0; c < KB; ++c) {
                v[c] = src[(k + c) * nxy + col];
                wv[c] = volz[k + c];
            }
#pragma unroll
            for (int c = 0; c < KB; ++c) acc += vxy * wv[c] * (double)v[c];
        }
        for (; k < q.k1; ++k) acc += vxy * volz[k] * (double)src[k * nxy + col];
    }
    const double s = wg_sum<256>(acc, red);
    if (threadIdx.x == 0) I.part[lb] = s;
}

}  // namespace tdgl
