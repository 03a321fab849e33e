// k_adj.hip -- kernels of the adjoint (reverse-mode) derivative of the
// time-averaged voltage with respect to eps(r).
//
// One implicit step maps (psi^-, mu^-, K^-) to (psi, mu, K): the
// Crank-Nicolson solve M psi = b of Sec. 3.1, J_av of Sec. 3.1.1, the K
// update of Eq. K_ODE and the Poisson solve of Sec. 3.2.  Its reverse, for a
// real loss L and complex adjoints zbar = dL/dRe z + i dL/dIm z:
//   fbar   = W G(W^-1 mubar)                  (Delta_h is W-self-adjoint)
//   psibar += -i fbar NS(psi) + i W NS(W^-1 fbar psi)
//   Kbar   += sum fbar dIm[psi^* NS psi]/dK,  Ebar = dt Kbar + dL/dE,
//   Jbar = -Ebar,  psibar += -i Jbar T psi / (N hx),  Kbar += Jbar dJ/dK
//   lambda = M^-H psibar, solved as M~ nu = W^-1 psibar with M~ = conj(diag)
//            - (ht/2) NS (the forward Jacobi sweep with other b/M, (ht/2)/M)
//   epsbar += (ht/2) Re[conj(lambda)(psi^- + psi)]
//   mubar^- = (u ht/2) Im[conj(lambda)(psi^- + psi)]
//   Kbar   += (ht/2) Re sum conj(lambda) dNS/dK (psi^- + psi)
//   psibar^- = conj(alpha) lambda + beta conj(lambda) + (ht/2) W L(W^-1 lambda)
// with alpha = 1 + (ht/2)(eps - i u mu^-) - ht |psi^-|^2 - (ht/2) conj(psi^-) psi
// and  beta  = -(ht/2) psi^-^2 - (ht/2) psi^- psi   (|psi^-|^2 psi^- is not
// holomorphic, hence the conj(lambda) term).  Sums over x edges use
// summation by parts so that every K term is a sum over edges (m, m+x).
// The kernels act on instance 0 of a one-instance context; flat kernels use
// a grid-stride loop over the nodes, and their per-block partials are summed
// by every work-group of the kernel that needs the sum (a launch of one
// work-group for that takes as long as a pass over a small grid).  A reverse
// step is four passes around the Poisson and the Jacobi solve, each with the
// neighbour sums it needs made from the caches: at the sizes of a gradient
// run (10^4 to 10^6 nodes) a pass is a chain of memory latencies of 3 to 8 us,
// whatever it computes, and one kernel per term made 21 of them (a gradient
// run of 24 steps at 72 x 60 x 10 6.5 ms, now 5.5; of 40 steps at 128 x 128 x
// 32 18.0, now 16.2; of 3 steps at 1024 x 512 x 64 24.1, now 20.4, where what
// counts are the neighbour sums no longer written and read back).
#include "kernels.h"
#include "stencil.h"

namespace tdgl {

__device__ __forceinline__ void node_ijk(const Inst &I, int m, int &i, int &j, int &k) {
    i = m % I.nx;
    const int r = m / I.nx;
    j = r % I.ny;
    k = r / I.ny;
}

__device__ __forceinline__ float node_wm(const Inst &I, int m) {
    int i, j, k;
    node_ijk(I, m, i, j, k);
    return node_w(I, i, j, k);
}

#define FLAT_LOOP(m) \
    for (int m = blockIdx.x * blockDim.x + threadIdx.x; m < I.N; m += gridDim.x * blockDim.x)

// State save / restore.  raw = 1 (checkpoints): psi, mu as stored and
// dK[0] = K, dK[1] = weighted mean of mu, dK[2] = step counter (it keys the
// Langevin draws), so that a restored step replays bit for bit.  raw = 0 (states the reverse sweep reads): mu with its
// weighted mean removed, as the step uses it, and dK[0] = K.  elog (null: not
// wanted): the last step's E.
__global__ void k_adj_save(const Inst *__restrict__ insts, float2 *dpsi, float *dmu, double *dK, int raw,
                           double *elog) {
    const Inst &I = insts[0];
    const float2 *psi = I.psi[I.st->cur];
    const float mean = raw ? 0.f : (float)I.st->mu_mean;
    FLAT_LOOP(m) {
        dpsi[m] = psi[m];
        dmu[m] = I.mu[m] - mean;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        dK[0] = I.st->K;
        if (elog) *elog = I.st->E_last;
        if (raw) {
            dK[1] = I.st->mu_mean;
            dK[2] = I.st->n;  // the step counter keys the Langevin draws of the replay
        }
    }
}

// Restores a raw = 1 save.
__global__ void k_adj_load(const Inst *__restrict__ insts, const float2 *spsi, const float *smu,
                           const double *sK) {
    const Inst &I = insts[0];
    float2 *psi = I.psi[I.st->cur];
    FLAT_LOOP(m) {
        psi[m] = spsi[m];
        I.mu[m] = smu[m];
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        I.st->K = sK[0];
        I.st->mu_mean = sK[1];
        I.st->n = sK[2];
    }
}

__global__ void k_adj_logE(const Inst *__restrict__ insts, double *Elog, int n) {
    if (threadIdx.x == 0) Elog[n] = insts[0].st->E_last;
}

// Vbar = (1/W) sum_{n = wb}^{nsteps-1} E_n, summed in step order by one
// thread (the same additions, in the same order, as a sequential host loop).
__global__ void k_adj_vbar(const double *Elog, int wb, int nsteps, double *vbar) {
    if (threadIdx.x != 0 || blockIdx.x != 0) return;
    double acc = 0.0;
    for (int n = wb; n < nsteps; ++n) acc += Elog[n];
    *vbar = acc / (double)(nsteps - wb);
}

__global__ void k_adj_zero(AdjState *adj) {
    if (threadIdx.x == 0) { adj->Kbar[0] = 0.0; adj->Kbar[1] = 0.0; adj->scale = 1.0; }
}

// Poisson transpose, right side f = W^-1 mubar, for the multigrid: the
// iterative solve starts from zero so that the result does not depend on what
// the buffer held.  (The spectral solve reads f where it is.)
__global__ void k_adj_prep_f(const Inst *__restrict__ insts, const float *f) {
    const Inst &I = insts[0];
    FLAT_LOOP(m) {
        I.f[m] = f[m];
        I.mu[m] = 0.f;
    }
}

// x links at K_n into uxn and at K_{n-1} into the instance's table (and that K
// into its state).
__global__ void k_adj_links(const Inst *__restrict__ insts, const double *Kn, const double *Km, float2 *uxn) {
    const Inst &I = insts[0];
    const double kn = *Kn, km = *Km, Bz = I.st->Bz;
    const double yref = link_yref(I, I.st);
    if (blockIdx.x == 0 && threadIdx.x == 0) I.st->K = km;
    for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < I.ny; j += gridDim.x * blockDim.x) {
        const double yb = j * I.hy - yref;
        uxn[j] = expi(I.hx * (kn + Bz * yb));
        I.ux[j] = expi(I.hx * (km + Bz * yb));
    }
}

// Neighbours of node m = (i, j, k) on a grid with periodic x: their flat
// indices in the order x-, x+, y-, y+, z-, z+ (an open face's ghost is the
// inner neighbour; a z neighbour that does not exist is the node itself).
struct AdjNb {
    int n[6];
    bool zm, zp;
};
__device__ __forceinline__ AdjNb adj_nb(const Inst &I, int m, int i, int j, int k) {
    const int nx = I.nx, ny = I.ny, nz = I.nz, nxy = nx * ny;
    AdjNb b;
    b.n[0] = i == 0 ? m + (nx - 1) : m - 1;
    b.n[1] = i == nx - 1 ? m - (nx - 1) : m + 1;
    const int lo = I.per[1] ? m + (ny - 1) * nx : (ny >= 2 ? m + nx : m);
    const int hi = I.per[1] ? m - (ny - 1) * nx : (ny >= 2 ? m - nx : m);
    b.n[2] = j == 0 ? lo : m - nx;
    b.n[3] = j == ny - 1 ? hi : m + nx;
    b.zm = k > 0 || I.per[2];
    b.zp = k < nz - 1 || I.per[2];
    b.n[4] = k > 0 ? m - nxy : (I.per[2] ? m + (nz - 1) * nxy : m);
    b.n[5] = k < nz - 1 ? m + nxy : (I.per[2] ? m - (nz - 1) * nxy : m);
    return b;
}

// Neighbour sum NS of a field with the values v at the neighbours: the wrap
// phases and ghosts of cell_src(), then nsum().
template <bool YZ>
__device__ __forceinline__ float2 adj_ns(const Inst &I, const AdjNb &b, int i, int j, int k, float2 ux, float2 *v) {
    if (j == 0 || j == I.ny - 1) {
        const float2 ph = I.P[k * I.nx + i], zero = make_float2(0.f, 0.f);
        if (j == 0) v[2] = I.per[1] ? xcmul(ph, v[2]) : (I.ny >= 2 ? v[2] : zero);
        if (j == I.ny - 1) v[3] = I.per[1] ? xcmulc(ph, v[3]) : (I.ny >= 2 ? v[3] : zero);
    }
    if (YZ) {
        ux = xcmul(ux, I.wz[k]);
        if (I.per[2]) {  // the seam phase of a periodic z axis
            const float2 zs = I.zs[i];
            if (k == 0) v[4] = xcmul(zs, v[4]);
            if (k == I.nz - 1) v[5] = xcmulc(zs, v[5]);
        }
    }
    return nsum(ux, I.uz[j], v[0], v[1], v[2], v[3], v[4], v[5], b.zm, b.zp, I.cx, I.cy, I.cz);
}

// Sums of NS arrays of n <= ADJ_GROUPS partials over a 256-thread work-group, in a
// fixed order, to all its threads.
template <int NS>
__device__ __forceinline__ void adj_sums(const double *const *part, int n, double *s) {
    __shared__ double red[NS][4];
    constexpr int C = ADJ_GROUPS / 256;
#pragma unroll
    for (int q = 0; q < NS; ++q) {
        double v[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int t = (int)threadIdx.x + c * 256;
            v[c] = t < n ? part[q][t] : 0.0;
        }
        s[q] = 0.0;
#pragma unroll
        for (int c = 0; c < C; ++c) s[q] += v[c];
    }
#pragma unroll
    for (int q = 0; q < NS; ++q) {
        for (int o = 32; o > 0; o >>= 1) s[q] += __shfl_xor(s[q], o, 64);
        if ((threadIdx.x & 63) == 0) red[q][threadIdx.x >> 6] = s[q];
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NS; ++q) s[q] = ((red[q][0] + red[q][1]) + red[q][2]) + red[q][3];
}

// Reverse of the Poisson right side, links at K_n, with mu the Poisson
// transpose's output and g = W^-1 fbar psi = (mu - mean) psi:
//   psibar += -i fbar NS(psi) + i W NS(g);
// partials of sum_m (fbar_m - fbar_{m+x}) Re[conj(psi_m) U_j psi_{m+x}] with U
// at K_n (part[0..]) and, for J_av, of sum Re[conj(psi_m) U_j psi_{m+x}] with
// U at K_{n-1} (part[G..], G work-groups in all four passes).
template <bool YZ>
__global__ __launch_bounds__(256) void k_adj_f(const Inst *__restrict__ insts, float2 *psibar, const float2 *psin,
                                               const float2 *uxn, double *part) {
    __shared__ double red[4];
    const Inst &I = insts[0];
    const float mean = (float)I.st->mu_mean;
    double acc = 0.0, accj = 0.0;
    FLAT_LOOP(m) {
        int i, j, k;
        node_ijk(I, m, i, j, k);
        const AdjNb b = adj_nb(I, m, i, j, k);
        float2 p[6], g[6];
        float mu[6];
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            p[q] = psin[b.n[q]];
            mu[q] = I.mu[b.n[q]];
        }
        const float2 pc = psin[m], pb = psibar[m];
        const float muc = I.mu[m];
        const float2 un = uxn[j], um = I.ux[j], wz = I.wz[k];
#pragma unroll
        for (int q = 0; q < 6; ++q) g[q] = cscale(mu[q] - mean, p[q]);
        const float2 px = p[1];
        const float w = node_w(I, i, j, k);
        const float fb = w * (muc - mean);
        const float2 a = adj_ns<YZ>(I, b, i, j, k, un, p), c = adj_ns<YZ>(I, b, i, j, k, un, g);
        // -i fb a + i w c
        psibar[m] = cadd(pb, make_float2(fb * a.y - w * c.y, -fb * a.x + w * c.x));
        const float fb1 = node_w(I, (i == I.nx - 1) ? 0 : i + 1, j, k) * (mu[1] - mean);
        const float2 upn = cmul(xcmul(un, wz), px), upm = cmul(xcmul(um, wz), px);
        acc += (double)(fb - fb1) * (double)(pc.x * upn.x + pc.y * upn.y);
        accj += (double)(pc.x * upm.x + pc.y * upm.y);
    }
    const double s = wg_sum<256>(acc, red), sj = wg_sum<256>(accj, red);
    if (threadIdx.x == 0) {
        part[blockIdx.x] = s;
        part[gridDim.x + blockIdx.x] = sj;
    }
}

// The K update's reverse from the partials (part[2 G ..]: those of the
// reverse step before, have2),
//   Kbar += (ht/2) S2 / hx;  Kbar += S0 / hx;  Jbar = -(dt Kbar + ew);
//   Kbar += Jbar S1 / N   (from adj->Kbar[kp] to adj->Kbar[kp ^ 1]),
// then psibar += -i Jbar (T psi) / (N hx) and partial maxima of |psibar| / w
// (part[3 G ..]).
__global__ __launch_bounds__(256) void k_adj_jterm(const Inst *__restrict__ insts, float2 *psibar,
                                                   const float2 *psin, double *part, int have2, int kp, double ew,
                                                   AdjState *adj) {
    __shared__ double red[4];
    const Inst &I = insts[0];
    const double *src[3] = {part, part + gridDim.x, part + 2 * gridDim.x};
    double S[3];
    adj_sums<3>(src, (int)gridDim.x, S);
    double Kbar = adj->Kbar[kp];
    if (have2) Kbar += (double)I.ht2 * S[2] / I.hx;
    Kbar += S[0] / I.hx;
    const double Jbar = -(I.dt * Kbar + ew);
    if (blockIdx.x == 0 && threadIdx.x == 0) adj->Kbar[kp ^ 1] = Kbar + Jbar * S[1] / (double)I.N;
    const float c = (float)(-Jbar / ((double)I.N * I.hx));
    double mx = 0.0;
    FLAT_LOOP(m) {
        int i, j, k;
        node_ijk(I, m, i, j, k);
        const int mp = (i == I.nx - 1) ? m - (I.nx - 1) : m + 1;
        const int mm = (i == 0) ? m + (I.nx - 1) : m - 1;
        const float2 u = xcmul(I.ux[j], I.wz[k]);
        const float2 t = csub(cmul(u, psin[mp]), cmulc(u, psin[mm]));
        // c * (i t)
        const float2 pb = cadd(psibar[m], make_float2(-c * t.y, c * t.x));
        psibar[m] = pb;
        mx = fmax(mx, (double)(sqrtf(cabs2(pb)) / node_w(I, i, j, k)));
    }
    for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o, 64));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
    __syncthreads();
    if (threadIdx.x == 0) part[3 * gridDim.x + blockIdx.x] = fmax(fmax(red[0], red[1]), fmax(red[2], red[3]));
}

// Adjoint system of step n: M~ nu = W^-1 psibar / scale with M from
// (psi^-, mu^-, eps) and scale the largest of the partial maxima (1 if 0).  Writes b/M~ and (ht/2)/M~.  The solve starts warm
// from the previous reverse steps' solutions: lamW holds scale' nu' of the
// last one (zero before the first) and lamW_old that of the one before, so
// nu^(0) = lamW / scale, or, with extrap, the linear extrapolation
// (2 lamW - lamW_old) / scale in reverse time (about a third fewer sweeps
// at 128 x 128 x 32; the stop rule is unchanged).  No sweep has
// produced that iterate, so it is stored as iterate 1 and convergence row 0
// is marked open (+inf): sweep 1 then measures the residual of nu^(0) and
// the solve proceeds as usual, one iteration index later.
__global__ __launch_bounds__(256) void k_adj_assemble(const Inst *__restrict__ insts, const float2 *psibar,
                                                      const float2 *psim, const float *mum,
                                                      const float2 *lamW, const float2 *lamW_old, int extrap,
                                                      const double *part, AdjState *adj) {
    __shared__ float red[4];
    __shared__ double mred[4];
    const Inst &I = insts[0];
    double mx = 0.0;
    for (int t = threadIdx.x; t < (int)gridDim.x; t += 256) mx = fmax(mx, part[3 * gridDim.x + t]);
    for (int o = 32; o > 0; o >>= 1) mx = fmax(mx, __shfl_xor(mx, o, 64));
    if ((threadIdx.x & 63) == 0) mred[threadIdx.x >> 6] = mx;
    __syncthreads();
    mx = fmax(fmax(mred[0], mred[1]), fmax(mred[2], mred[3]));
    const double scale = mx > 0.0 ? mx : 1.0;
    if (blockIdx.x == 0 && threadIdx.x == 0) adj->scale = scale;
    const float inv_s = (float)(1.0 / scale);
    const float ht2 = I.ht2, S2 = I.S2, u = I.u;
    float2 *nu1 = I.psi[I.st->cur ^ 1];
    FLAT_LOOP(m) {
        const float2 p = psim[m];
        const float a2 = cabs2(p);
        const float e = I.eps[m], um = u * mum[m];
        // conj(M_mm) with M = 1 + ht/2 (|p|^2 + 2S + i u mu - eps)
        const float2 Mc = make_float2(1.f + ht2 * (a2 + S2 - e), -ht2 * um);
        const float inv = 1.f / cabs2(Mc);
        const float2 Mi = make_float2(Mc.x * inv, -Mc.y * inv);
        const float2 rhs = cscale(inv_s / node_wm(I, m), psibar[m]);
        const float2 bhv = cmul(rhs, Mi), dhv = cscale(ht2, Mi);
        I.bh[m] = bhv;
        I.dh[m] = dhv;
        if (I.edge) {
            // side copies for the two-sweep super-tiles
            const int x = (int)(m % I.nx), t = (int)(m / I.nx);
            int el, er;
            edge_slots(I, x, t % I.ny, t / I.ny, el, er);
            if (el >= 0) {
                I.edge[el] = bhv;
                I.edge[el + 1] = dhv;
            }
            if (er >= 0) {
                I.edge[er] = bhv;
                I.edge[er + 1] = dhv;
            }
        }
        const float2 w0 = lamW[m];
        float2 g = w0;
        if (extrap) {
            const float2 w1 = lamW_old[m];
            g = make_float2(2.f * w0.x - w1.x, 2.f * w0.y - w1.y);
        }
        nu1[m] = cscale(inv_s, g);
    }
    wg_max_to<256>(row_slot(I.res, I.rstride, 0, blockIdx.x), __int_as_float(0x7f800000), red);
}

// epsbar, f = W^-1 mubar^- (the next reverse step's Poisson right side) and
// psibar^- from lambda = W scale nu; lambda / W into lamW (the next reverse
// steps' warm start); partials (part[2 G ..]) of
//   Re[i sum_m (conj(lambda_m) U_j s_{m+x} - conj(lambda_{m+x} U_j) s_m)],
// s = psi^- + psi.
template <bool YZ>
__global__ __launch_bounds__(256) void k_adj_sources(const Inst *__restrict__ insts, float2 *psibar, float *f,
                                                     float *epsbar, const float2 *psim, const float2 *psin,
                                                     const float *mum, float2 *lamW, double *part,
                                                     const AdjState *adj) {
    __shared__ double red[4];
    const Inst &I = insts[0];
    const float s = (float)adj->scale;
    const float ht2 = I.ht2, u = I.u, S2 = I.S2;
    const float2 *nu = I.psi[I.st->cur];
    double acc = 0.0;
    FLAT_LOOP(m) {
        int i, j, k;
        node_ijk(I, m, i, j, k);
        const AdjNb b = adj_nb(I, m, i, j, k);
        float2 v[6];
#pragma unroll
        for (int q = 0; q < 6; ++q) v[q] = nu[b.n[q]];
        const float2 nc = nu[m], p = psim[m], q = psin[m], p1 = psim[b.n[1]], q1 = psin[b.n[1]];
        const float e = I.eps[m], mm = mum[m], eb = epsbar[m];
        const float2 ux = I.ux[j], wz = I.wz[k];
        const float w = node_w(I, i, j, k);
        const float2 lam1 = cscale(node_w(I, i == I.nx - 1 ? 0 : i + 1, j, k) * s, v[1]);
#pragma unroll
        for (int c = 0; c < 6; ++c) v[c] = cscale(s, v[c]);
        const float2 ns = adj_ns<YZ>(I, b, i, j, k, ux, v);
        const float2 lam = cscale(w * s, nc);
        const float2 sm = cadd(p, q);
        const float2 cl_s = cmulc(lam, sm);  // conj(lambda) * (psi^- + psi)
        epsbar[m] = eb + ht2 * cl_s.x;
        f[m] = (u * ht2 * cl_s.y) / w;
        const float a2 = cabs2(p), um = u * mm;
        // alpha = 1 + ht/2 (eps - i u mu) - ht |p|^2 - ht/2 conj(p) q
        const float2 cpq = cmulc(p, q);
        const float2 alpha = make_float2(1.f + ht2 * e - 2.f * ht2 * a2 - ht2 * cpq.x, -ht2 * um - ht2 * cpq.y);
        // beta = -ht/2 p^2 - ht/2 p q
        const float2 p2 = cmul(p, p), pq = cmul(p, q);
        const float2 beta = make_float2(-ht2 * (p2.x + pq.x), -ht2 * (p2.y + pq.y));
        const float2 t1 = cmulc(alpha, lam);                                  // conj(alpha) lambda
        const float2 t2 = cmul(beta, make_float2(lam.x, -lam.y));             // beta conj(lambda)
        const float2 lh = make_float2(w * ns.x - S2 * lam.x, w * ns.y - S2 * lam.y);
        psibar[m] = make_float2(t1.x + t2.x + ht2 * lh.x, t1.y + t2.y + ht2 * lh.y);
        lamW[m] = cscale(s, nc);
        const float2 uw = xcmul(ux, wz);
        const float2 a = cmulc(lam, cmul(uw, cadd(p1, q1)));  // conj(lambda_m) U s_{m+x}
        const float2 bb = cmulc(cmul(lam1, uw), sm);          // conj(lambda_{m+x} U) s_m
        // Re[i (a - bb)] = -(a - bb).y
        acc += -(double)(a.y - bb.y);
    }
    const double t = wg_sum<256>(acc, red);
    if (threadIdx.x == 0) part[2 * gridDim.x + blockIdx.x] = t;
}

template __global__ void k_adj_f<false>(const Inst *, float2 *, const float2 *, const float2 *, double *);
template __global__ void k_adj_f<true>(const Inst *, float2 *, const float2 *, const float2 *, double *);
template __global__ void k_adj_sources<false>(const Inst *, float2 *, float *, float *, const float2 *,
                                              const float2 *, const float *, float2 *, double *, const AdjState *);
template __global__ void k_adj_sources<true>(const Inst *, float2 *, float *, float *, const float2 *,
                                             const float2 *, const float *, float2 *, double *, const AdjState *);

#undef FLAT_LOOP

}  // namespace tdgl
