// k_blk.hip -- several Jacobi iterations per launch on small and mid-size
// grids (gfx950).
//
// On a grid of up to a few million nodes a sweep is not bound by HBM: the
// arrays stay in the last-level cache, and a z-marching work-group spends
// its life in a chain of dependent loads and barriers (32 x 32 x 16 nodes:
// 7.2 us a sweep for 0.5 MB).  Here a work-group takes a BX x BY x BZ block,
// loads psi^(l) of the block with an S-node halo into LDS at once, and makes
// S iterates from it: stage s computes psi^(l+s+1) on the block with a halo
// of S-1-s nodes, in place (the new values wait in registers across one
// barrier).  The halo's iterates are computed again by the neighbours; that
// work is cheap next to a launch and a load latency per sweep.
//
// A thread owns one (x, y) column of the block with its halo in every stage,
// so b/M and (ht/2)/M of its nodes are loaded once, ahead of the first
// stage, and stay in registers, as does all that depends on (x, y) only:
// links, boundary rules and LDS offsets.
//
// LDS holds the real node behind every slot (periodic images unphased); the
// boundary rules of Sec. 3.3 act where a stencil crosses the boundary: the
// quasi-periodic phase P between rows ny-1 and 0, the Neumann mirror node
// (times U^2 on an open x face).  Each value is the same function of the same
// operands as in the single-sweep kernel, so the iterates are bit-identical.
//
// FIRST: stage 0 is the assemble (b/M and (ht/2)/M are computed for the halo
// too, stored for the block), so one launch makes psi^(1) .. psi^(S).
#include "kernels.h"
#include "stencil.h"

#include <type_traits>

namespace tdgl {

namespace {

// Real index of position g in [-S, B + S) on an axis of n nodes (periodic:
// any wrap); -1: no such node (open axis).  n is uniform, so the division is
// skipped as a whole except on axes shorter than a block with its halo.
template <int REACH>
__device__ __forceinline__ int real_index(int g, int n, bool per) {
    if (!per) return ((unsigned)g < (unsigned)n) ? g : -1;
    if (n < REACH) {
        const int r = g % n;
        return r < 0 ? r + n : r;
    }
    return g < 0 ? g + n : (g >= n ? g - n : g);
}

// nsum() with the z term selected rather than branched to, so that the planes
// of a column can be scheduled together; the same operations on the same
// operands.
__device__ __forceinline__ float2 nsum_sel(float2 ux, float2 uz, float2 xm, float2 xp, float2 ym, float2 yp,
                                           float2 zmv, float2 zpv, bool zm, bool zp, float cx, float cy, float cz) {
#pragma clang fp contract(off)
    const float2 a = xcmul(uz, zpv), b = xcmulc(uz, zmv);
    const float2 ab = xcadd(a, b);
    const float2 one = zp ? a : b;
    float2 zt = make_float2(2.f * one.x, 2.f * one.y);
    if (zm && zp) zt = ab;
    if (!zm && !zp) zt = make_float2(0.f, 0.f);
    const float2 xt = xcadd(xcmul(ux, xp), xcmulc(ux, xm));
    const float2 yt = xcadd(yp, ym);
    return make_float2(__builtin_fmaf(cx, xt.x, __builtin_fmaf(cy, yt.x, cz * zt.x)),
                       __builtin_fmaf(cx, xt.y, __builtin_fmaf(cy, yt.y, cz * zt.y)));
}

}  // namespace

// One pass of ns <= S iterates from psi^(l) (FIRST: l = 0 and the assemble).
// prefix: blocks per instance.  np: rows the previous pass wrote (l - np ..
// l - 1); the pass hands them to the host and exits when one of them met the
// tolerance, when that pass exited (rows never written read 0) or when the
// instance's cap is reached.  Pass number `pass` reads psi[cur ^
// (pass & 1)] and writes the other buffer.  l = -1: timing (psi[cur] to the
// spare buffer, nothing recorded); l = -2: the corrective pass of st->fix
// iterates from psi[cur ^ 1] into psi[cur] (see k_solve_finalize).
template <int BX, int BY, int BZ, int S, int HZ, int MODE, bool YZ>
__global__ __launch_bounds__(blk_threads(BX, BY, S)) void k_blk(const Inst *__restrict__ insts,
                                                                const int *__restrict__ prefix, int ninst, int l,
                                                                int ns, int np, int pass, unsigned long long *pub,
                                                                unsigned seq) {
    constexpr bool FIRST = MODE != MODE_SWEEP;
    constexpr int LX = BX + 2 * S, LY = BY + 2 * S, LZ = BZ + 2 * HZ, LXY = LX * LY;
    // planes that the first stage updates: with a z halo all but the outer
    // two, without one (HZ = 0: the block holds all of an open z axis) all
    constexpr int KA = HZ ? 1 : 0, KB = HZ ? LZ - 1 : LZ;
    constexpr int NT = blk_threads(BX, BY, S), NW = NT / 64;
    __shared__ float2 la[LZ][LXY];
    __shared__ float red[S][NW];

    const int b = xcd_remap(blockIdx.x, gridDim.x);
    const int ii = find_inst(prefix, ninst, b);
    const Inst &I = insts[ii];
    DevState *st = I.st;
    const int nx = I.nx, ny = I.ny, nz = I.nz;
    const bool timing = l == -1, fixp = !FIRST && l == -2;
    const int cur = st->cur;
    int q = b - prefix[ii];
    const bool first_block = q == 0;
    if (fixp) {
        ns = st->fix;
        if (ns <= 0) return;
    } else if (!FIRST && !timing) {
        // an instance at its cap has no iterate left to make, but rows below
        // the cap row that the host waits for while others iterate
        const bool capped = l >= I.max_iter;
        if (capped && !(pub && first_block)) return;
        // the two halves of a wavefront read two rows at a time
        bool done = false;
        for (int r = 0; r < np; r += 2) {
            const int h = (int)((threadIdx.x >> 5) & 1);
            const int row = l - np + min(r + h, np - 1);
            const float v = row_max_half(I.res, I.rstride, row);
            if (pub && first_block && (threadIdx.x & 31) == 0 && threadIdx.x < 64 && r + h < np)
                publish(pub + (size_t)row * ninst + ii, seq, v);
            done = done || __ballot(v < I.tol) != 0;
        }
        if (done || capped) return;
    }
    const int tx = (nx + BX - 1) / BX, ty = (ny + BY - 1) / BY;
    const int bx = q % tx;
    q /= tx;
    const int by = q % ty, bz = q / ty;
    const int x0 = bx * BX, y0 = by * BY, z0 = bz * BZ;
    const bool xper = I.per[0] != 0, yper = I.per[1] != 0, zper = I.per[2] != 0;
    const unsigned NXY = (unsigned)nx * (unsigned)ny;
    const int xs = timing ? 0 : (fixp ? 1 : (pass & 1));
    const gf2 *__restrict__ src = (const gf2 *)I.psi[cur ^ xs];
    gf2 *__restrict__ dst = (gf2 *)I.psi[cur ^ xs ^ 1];
    gf2 *bhp = (gf2 *)I.bh, *dhp = (gf2 *)I.dh;

    // this thread's column, slot (ci, cj) of the block with its halo
    const int tid = (int)threadIdx.x;
    const int ci = tid % LX, cj = tid / LX;
    const int gx = x0 - S + ci, gy = y0 - S + cj;
    const int rx = real_index<BX + S>(gx, nx, xper), ry = real_index<BY + S>(gy, ny, yper);
    const bool col = tid < LXY && (rx | ry) >= 0;
    const bool own = col && ci >= S && ci < S + BX && cj >= S && cj < S + BY && gx < nx && gy < ny;
    // it takes part in the stages s < ring
    const int ring = col ? min(min(ci, LX - 1 - ci), min(cj, LY - 1 - cj)) : 0;
    const unsigned so = col ? (unsigned)(ry * nx + rx) : 0u;
    // real planes of the column's slots (uniform); a slot without one reads a
    // real plane and is never stored
    int rz[LZ];
    bool vz[LZ];
#pragma unroll
    for (int k = 0; k < LZ; ++k) {
        const int p = real_index<BZ + HZ>(z0 - HZ + k, nz, zper);
        vz[k] = p >= 0;
        rz[k] = max(p, 0);
    }
    // every load is issued before the first value is used: psi^(l), then
    // b/M and (ht/2)/M (or eps and mu for the assemble), the phases
    float2 v[LZ], bh[LZ], dh[LZ];
    float ep[LZ], mu[LZ];
#pragma unroll
    for (int k = 0; k < LZ; ++k) v[k] = ld2(src, (unsigned)rz[k] * NXY + so);
#pragma unroll
    for (int k = KA; k < KB; ++k) {
        const unsigned m = (unsigned)rz[k] * NXY + so;
        if (FIRST) {
            ep[k] = ((const gf1 *)I.eps)[m];
            mu[k] = I.driven ? float(((const gf1 *)I.mu)[m]) : 0.f;
        } else {
            bh[k] = ld2(bhp, m);
            dh[k] = ld2(dhp, m);
        }
    }
    const float mu_mean = (FIRST && I.driven) ? (float)st->mu_mean : 0.f;
    const int row = col ? ry : 0;
    const float2 ux = ld2((const gf2 *)I.ux, row), uz = ld2((const gf2 *)I.uz, row);
    // boundary rules of the column: bits 0/1 open-x ghost factor on x-/x+,
    // 2/3 phase P (conj P) on y-/y+, 4 no x neighbours, 5 no y neighbours
    int xmo = -1, xpo = 1, ymo = -LX, ypo = LX;
    int rule = 0;
    if (!xper) {
        if (nx == 1) rule |= 16;
        else if (rx == 0) { xmo = 1; rule |= 1; }
        if (nx > 1 && rx == nx - 1) { xpo = -1; rule |= 2; }
    }
    if (yper) {
        if (ry == 0) rule |= 4;
        if (ry == ny - 1) rule |= 8;
    } else {
        if (ny == 1) rule |= 32;
        else if (ry == 0) ymo = LX;
        if (ny > 1 && ry == ny - 1) ypo = -LX;
    }
    if (ring == 0) rule = 0;  // halo column: only its psi^(l) is used
    const bool anyrule = __ballot(rule != 0) != 0;
    float2 ph[LZ], wz[LZ];
    if (__ballot((rule & 12) != 0) != 0) {
#pragma unroll
        for (int k = KA; k < KB; ++k) ph[k] = ld2((const gf2 *)I.P, (unsigned)(rz[k] * nx + max(rx, 0)));
    }
    if (YZ) {
#pragma unroll
        for (int k = KA; k < KB; ++k) wz[k] = ld2((const gf2 *)I.wz, (unsigned)rz[k]);
    }
    const float2 u2 = xcmul(ux, ux), u2c = make_float2(u2.x, -u2.y);
    const float cx = I.cx, cy = I.cy, cz = I.cz, ht2 = I.ht2, S2 = I.S2, u = I.u;
    const bool noise = (MODE == MODE_FIRSTN) && I.zeta_max > 0.f;
    const unsigned long long nstep = noise ? (unsigned long long)st->n : 0ull;
    const int s0 = S - ns;  // fewer iterates: the outer halo's stages are left out
    float rmax[S];
#pragma unroll
    for (int s = 0; s < S; ++s) rmax[s] = 0.f;
    const bool inx = tid < LXY;
    if (inx) {
#pragma unroll
        for (int k = 0; k < LZ; ++k) la[k][tid] = v[k];
    }
    __syncthreads();
    // stage s of the column: v[k] of psi^(l+s) becomes psi^(l+s+1)
    auto stage = [&](int s, bool asmb, auto ruled) __attribute__((always_inline)) {
        float2 zm1 = HZ ? v[s] : make_float2(0.f, 0.f);
#pragma unroll
        for (int k = KA + (HZ ? s : 0); k < KB - (HZ ? s : 0); ++k) {
            const float2 *L = &la[k][tid];
            float2 xm = L[xmo], xp = L[xpo], ym = L[ymo], yp = L[ypo];
            float2 uxk = ux;
            if (YZ) uxk = xcmul(ux, wz[k]);
            if constexpr (decltype(ruled)::value) {
                float2 fm = u2, fp = u2c;
                if (YZ) {
                    const float2 w2 = xcmul(wz[k], wz[k]);
                    fm = xcmul(u2, w2);
                    fp = xcmul(u2c, make_float2(w2.x, -w2.y));
                }
                if (rule & 1) xm = xcmul(fm, xm);
                if (rule & 2) xp = xcmul(fp, xp);
                if (rule & 4) ym = xcmul(ph[k], ym);
                if (rule & 8) yp = xcmulc(ph[k], yp);
                if (rule & 16) xm = xp = make_float2(0.f, 0.f);
                if (rule & 32) ym = yp = make_float2(0.f, 0.f);
            }
            const float2 c = v[k];
            const int p = rz[k];
            const bool zm = (p > 0) || zper, zp = (p < nz - 1) || zper;
            const float2 nsv = nsum_sel(uxk, uz, xm, xp, ym, yp, zm1, k + 1 < LZ ? v[k + 1 < LZ ? k + 1 : k] : c, zm, zp, cx, cy, cz);
            // the block's own nodes: their residual counts, and the assemble
            // stores their b/M and (ht/2)/M
            const bool mine = own && k >= HZ && k < HZ + BZ && z0 + (k - HZ) < nz;
            const unsigned m = (unsigned)p * NXY + so;
            float r2;
            float2 nw;
            if (FIRST && asmb) {
                const float2 zz = noise ? langevin2(I, m, nstep) : make_float2(0.f, 0.f);
                assemble_node(c, ep[k], u * (mu[k] - mu_mean), nsv, S2, ht2, noise, zz, bh[k], dh[k], nw, r2);
                if (mine) {
                    st2(bhp, m, bh[k]);
                    st2(dhp, m, dh[k]);
                }
            } else {
                nw = jacobi(bh[k], dh[k], nsv);
                r2 = resid2(nw, c, dh[k], ht2);
            }
            if (mine) rmax[s] = (r2 > rmax[s] || r2 != r2) ? r2 : rmax[s];
            if (s == S - 1 && mine) st2(dst, m, nw);
            zm1 = c;
            v[k] = nw;
        }
    };
#pragma unroll
    for (int s = 0; s < S; ++s) {
        if (s < s0) continue;
        const bool act = ring > s;
        if (act) {
            if (anyrule) stage(s, s == s0, std::true_type{});
            else stage(s, s == s0, std::false_type{});
        }
        if (s < S - 1) {
            __syncthreads();
            if (act) {
#pragma unroll
                for (int k = KA + (HZ ? s : 0); k < KB - (HZ ? s : 0); ++k)
                    if (vz[k]) la[k][tid] = v[k];
            }
            __syncthreads();
        }
    }
    if (timing || fixp) return;
    // max |r|^2 of every stage's input iterate
#pragma unroll
    for (int s = 0; s < S; ++s) {
        unsigned m = __float_as_uint(rmax[s]);
        for (int o = 32; o > 0; o >>= 1) {
            const unsigned w = __shfl_xor(m, o, 64);
            m = w > m ? w : m;
        }
        if ((threadIdx.x & 63) == 0) red[s][threadIdx.x >> 6] = __uint_as_float(m);
    }
    __syncthreads();
    if (tid < ns && l + tid < I.max_iter) {
        unsigned m = 0;
        for (int w = 0; w < NW; ++w) {
            const unsigned x = __float_as_uint(red[s0 + tid][w]);
            m = x > m ? x : m;
        }
        atomicMax(row_slot(I.res, I.rstride, l + tid, b), m);
    }
}

#define TDGL_BLK(BX, BY, BZ, S, HZ, MODE, YZ)                                                                       \
    template __global__ void k_blk<BX, BY, BZ, S, HZ, MODE, YZ>(const Inst *, const int *, int, int, int, int, int, \
                                                            unsigned long long *, unsigned);
#define TDGL_BLK_T(BX, BY, BZ, S, HZ)             \
    TDGL_BLK(BX, BY, BZ, S, HZ, MODE_SWEEP, false)  \
    TDGL_BLK(BX, BY, BZ, S, HZ, MODE_SWEEP, true)   \
    TDGL_BLK(BX, BY, BZ, S, HZ, MODE_FIRST, false)  \
    TDGL_BLK(BX, BY, BZ, S, HZ, MODE_FIRST, true)   \
    TDGL_BLK(BX, BY, BZ, S, HZ, MODE_FIRSTN, false) \
    TDGL_BLK(BX, BY, BZ, S, HZ, MODE_FIRSTN, true)
TDGL_BLK_VARIANTS(TDGL_BLK_T)
#undef TDGL_BLK_T
#undef TDGL_BLK

}  // namespace tdgl
