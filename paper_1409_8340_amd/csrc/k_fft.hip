// k_fft.hip -- direct spectral solve of the scalar-potential Poisson equation
// on gfx950 for a periodic x, periodic y, open z box.
//
// The 7-point operator of Sec. 3.2 separates: discrete Fourier modes
// diagonalise its x and y parts (periodic wrap), leaving for every
// (kx, ky) a real tridiagonal system along z (Neumann reflection at the
// open faces):
//     c_z mu_{k-1} - (lam_xy + 2 c_z) mu_k + c_z mu_{k+1} = f^_k,
// with the inner neighbour doubled on the two face rows and
//     lam_xy = c_x (2 - 2 cos(2 pi kx / nx)) + c_y (2 - 2 cos(2 pi ky / ny)).
// Steps: real-to-complex FFT along x (two rows per complex transform), FFT
// along y, the z systems by Thomas' algorithm with precomputed pivots in
// double precision (its two sweeps evaluated as prefix scans of affine maps
// across a wavefront), inverse FFT along y, complex-to-real inverse along x.
// The inverse x pass also sums the weighted mean of mu.  Where a few kx planes
// (all y and z) fit a work-group's LDS, for every spectral instance of the
// context, the y transforms and the z systems are one kernel (k_fft_yz) on a
// half spectrum stored kx-major; if all of them have an even ny, the forward x
// pass of a time step then makes the right side f = Im[psi^* NS psi] from psi
// itself (otherwise k_stencil<MODE_RHS> does).  The (0, 0) system
// is singular (the constant mode); its right side is projected onto the
// range (zero weighted mean) and its solution shifted to zero weighted mean,
// which fixes sum_m w_m mu_m = 0 for the whole grid.
//
// The FFTs are Stockham auto-sort transforms in LDS: each pass reads all of
// a thread's butterfly inputs into registers, synchronises, and writes the
// outputs to their sorted positions, so a single LDS buffer suffices.
#include "kernels.h"
#include "stencil.h"

namespace tdgl {

namespace {

// In-register DFT of size R (sign -1 forward, +1 inverse).
template <int R>
__device__ __forceinline__ void dft(float2 *v, float sign);

template <>
__device__ __forceinline__ void dft<2>(float2 *v, float) {
    const float2 a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
}

template <>
__device__ __forceinline__ void dft<3>(float2 *v, float sign) {
    const float c1 = -0.5f, s1 = sign * 0.86602540378443864676f;
    const float2 a = v[0], b = v[1], c = v[2];
    const float2 t = cadd(b, c), d = csub(b, c);
    v[0] = cadd(a, t);
    const float2 m = make_float2(a.x + c1 * t.x, a.y + c1 * t.y);
    // i * s1 * d
    const float2 j = make_float2(-s1 * d.y, s1 * d.x);
    v[1] = cadd(m, j);
    v[2] = csub(m, j);
}

template <>
__device__ __forceinline__ void dft<4>(float2 *v, float sign) {
    const float2 a = v[0], b = v[1], c = v[2], d = v[3];
    const float2 s0 = cadd(a, c), s1 = csub(a, c), s2 = cadd(b, d), s3 = csub(b, d);
    // i * sign * s3
    const float2 j = make_float2(-sign * s3.y, sign * s3.x);
    v[0] = cadd(s0, s2);
    v[2] = csub(s0, s2);
    v[1] = cadd(s1, j);
    v[3] = csub(s1, j);
}

template <>
__device__ __forceinline__ void dft<5>(float2 *v, float sign) {
    const float c1 = 0.30901699437494742410f, c2 = -0.80901699437494742410f;
    const float s1 = sign * 0.95105651629515357212f, s2 = sign * 0.58778525229247312917f;
    const float2 a = v[0];
    const float2 t1 = cadd(v[1], v[4]), t2 = cadd(v[2], v[3]);
    const float2 d1 = csub(v[1], v[4]), d2 = csub(v[2], v[3]);
    v[0] = make_float2(a.x + t1.x + t2.x, a.y + t1.y + t2.y);
    const float2 m1 = make_float2(a.x + c1 * t1.x + c2 * t2.x, a.y + c1 * t1.y + c2 * t2.y);
    const float2 m2 = make_float2(a.x + c2 * t1.x + c1 * t2.x, a.y + c2 * t1.y + c1 * t2.y);
    // i * (s1 d1 + s2 d2) and i * (s2 d1 - s1 d2)
    const float2 e1 = make_float2(s1 * d1.x + s2 * d2.x, s1 * d1.y + s2 * d2.y);
    const float2 e2 = make_float2(s2 * d1.x - s1 * d2.x, s2 * d1.y - s1 * d2.y);
    const float2 j1 = make_float2(-e1.y, e1.x), j2 = make_float2(-e2.y, e2.x);
    v[1] = cadd(m1, j1);
    v[4] = csub(m1, j1);
    v[2] = cadd(m2, j2);
    v[3] = csub(m2, j2);
}

constexpr int FFT_THREADS = FFT_XY_THREADS;  // threads of the y passes
constexpr int ZS_THREADS = 256;              // threads of the z solve (4 wavefronts)
constexpr int FFT_MAXPTS = FFT_MAXN;  // points per work-group of the y passes (all sequences)


// q = floor(t / d) for 0 <= t < 2^20 and 1 <= d <= 2^13, from a float
// reciprocal: (t + 1/2) / d stays at least 1/(2d) away from an integer,
// far more than the rounding of the product.
__device__ __forceinline__ int fdiv(int t, float inv_d) { return (int)(((float)t + 0.5f) * inv_d); }

// One Stockham pass of radix R over `nseq` sequences of length n stored in
// LDS at buf[s * sstride + e] (element e), by NT threads; MAXC bounds the
// points n * nseq.  Ns = product of the radices of the previous passes.
// tw[k] = exp(-2 pi i k / n) (conjugated for the inverse transform,
// sign = +1).
template <int R, int NT, int MAXC>
__device__ __forceinline__ void fft_pass(float2 *buf, int n, int Ns, int nseq, int sstride, const float2 *tw,
                                         float sign) {
    constexpr int MAXBF = (MAXC / R + NT - 1) / NT;
    const int nb = n / R;
    const int total = nb * nseq;
    const float inv_nb = 1.0f / (float)nb, inv_ns = 1.0f / (float)Ns;
    const int tstep = n / (Ns * R);
    float2 v[MAXBF][R];
    int dst[MAXBF];
#pragma unroll
    for (int i = 0; i < MAXBF; ++i) {
        const int t = threadIdx.x + i * NT;
        if (t < total) {
            const int s = fdiv(t, inv_nb), j = t - s * nb;
            const int jq = fdiv(j, inv_ns), jm = j - jq * Ns;
            const float2 *row = buf + s * sstride;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float2 a = row[j + r * nb];
                if (r == 0 || jm == 0) {
                    v[i][r] = a;
                } else {
                    float2 w = tw[jm * r * tstep];
                    w.y *= -sign;
                    v[i][r] = cmul(a, w);
                }
            }
            dft<R>(v[i], sign);
            dst[i] = s * sstride + jq * Ns * R + jm;
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < MAXBF; ++i) {
        const int t = threadIdx.x + i * NT;
        if (t < total) {
#pragma unroll
            for (int r = 0; r < R; ++r) buf[dst[i] + r * Ns] = v[i][r];
        }
    }
    __syncthreads();
}

// Full transform of nseq sequences in LDS (natural order in and out).
// P2: the length is a power of two (radices 4 and 2 only), which keeps the
// kernels small enough for two 1024-thread work-groups per CU.
template <bool P2, int NT, int MAXC>
__device__ __forceinline__ void fft_lds(float2 *buf, int n, const int *rad, int nrad, int nseq, int sstride,
                                        const float2 *tw, float sign) {
    int Ns = 1;
    for (int p = 0; p < nrad; ++p) {
        const int R = rad[p];
        if (R == 4) fft_pass<4, NT, MAXC>(buf, n, Ns, nseq, sstride, tw, sign);
        else if (P2 || R == 2) fft_pass<2, NT, MAXC>(buf, n, Ns, nseq, sstride, tw, sign);
        else if (R == 3) fft_pass<3, NT, MAXC>(buf, n, Ns, nseq, sstride, tw, sign);
        else fft_pass<5, NT, MAXC>(buf, n, Ns, nseq, sstride, tw, sign);
        Ns *= R;
    }
}

// fft_lds by a work-group of FFT_YZ_THREADS threads, up to FFT_YZ_BATCH points
// (whole sequences) at a time: all of FFT_YZ_PTS at once would spill the
// butterflies of radices 3 and 5.
template <bool P2>
__device__ __forceinline__ void fft_lds_batches(float2 *buf, int n, const int *rad, int nrad, int nseq, int sstride,
                                                const float2 *tw, float sign) {
    const int per = max(1, FFT_YZ_BATCH / n);
    for (int s = 0; s < nseq; s += per)
        fft_lds<P2, FFT_YZ_THREADS, FFT_YZ_BATCH>(buf + s * sstride, n, rad, nrad, min(per, nseq - s), sstride, tw,
                                                  sign);
}

// Coefficients of row k of the z system of column (kx, ky):
//   a_k mu_{k-1} + b_k mu_k + c_k mu_{k+1} = d_k.
// Face rows carry the doubled inner neighbour (Neumann reflection); the
// singular (0, 0) column has row 0 replaced by mu_0 = 0.
__device__ __forceinline__ void zrow(int k, int nz, double cz, bool singular, double &a, double &c) {
    if (nz == 1 || (singular && k == 0)) { a = 0.0; c = 0.0; return; }
    a = (k == 0) ? 0.0 : (k == nz - 1 ? 2.0 * cz : cz);
    c = (k == nz - 1) ? 0.0 : (k == 0 ? 2.0 * cz : cz);
}

}  // namespace

// Row pairs per work-group of the x passes: about FFT_X_PTS complex points
// (one pair of 1024-point rows), at least one pair, no more than a plane has.
__host__ __device__ int fft_x_pairs(int nx, int ny) {
    int p = FFT_X_PTS / nx;
    p = p < 1 ? 1 : (p > 32 ? 32 : p);
    const int h = (ny + 1) / 2;
    return p < h ? p : h;
}
// LDS of the x passes (complex elements): the rows (nx + 1 apart, so that
// reads down a column spread over the banks) and the twiddles.
__host__ __device__ int fft_x_lds(int nx, int ny) { return fft_x_pairs(nx, ny) * (nx + 1) + nx; }
// kx planes per work-group of k_fft_yz (0: they do not fit): about 1024
// points (one per thread), at most FFT_YZ_LDS complex elements with the padding of the columns
// and the twiddles.
__host__ __device__ int fft_yz_planes(int nx, int ny, int nz) {
    const int P = nx / 2 + 1;
    if (nx > FFT_X_PTS || (long)(ny + 1) * nz + ny > FFT_YZ_LDS || (long)ny * nz > FFT_YZ_PTS || ny > FFT_YZ_BATCH) return 0;
    int g = FFT_YZ_TARGET / (ny * nz);
    g = g < 1 ? 1 : (g > P ? P : g);
    return g;
}
__host__ __device__ int fft_yz_lds(int ny, int nz, int g) { return g * nz * (ny + 1) + ny; }
// Tiles of the y passes over an instance's columns (z, kx), P = nx/2 + 1
// per plane: a work-group holds at most FFT_MAXPTS points (and 1024
// columns).  Where a whole plane's P columns fit, a tile is G whole planes
// (as many as fit); otherwise each plane is cut into ntk tiles of about
// equal width.  Tiles start on a plane or at kx = j TK within one, so their
// rows start on the same 128-byte lines for every plane.
__host__ __device__ FftYPlan fft_y_plan(int nx, int ny, int nz) {
    const int P = nx / 2 + 1;
    int t = FFT_MAXPTS / ny;
    t = t < 1 ? 1 : (t > 1024 ? 1024 : t);
    FftYPlan q;
    if (t >= P) {
        q.G = t / P < nz ? t / P : nz;
        q.ntk = 1;
        q.TK = q.G * P;
    } else {
        q.G = 1;
        q.ntk = (P + t - 1) / t;
        q.TK = (P + q.ntk - 1) / q.ntk;
    }
    q.blocks = ((nz + q.G - 1) / q.G) * q.ntk;
    return q;
}
// LDS stride of the y passes' columns (complex elements).
__host__ __device__ int fft_y_stride(int ny) { return ny + 1; }
// Row pitch (complex elements) of the half spectrum: nx/2 + 1 rounded up to
// 16 elements, so that every row starts on a 128-byte line.
__host__ __device__ int fft_pitch(int nx) { return (nx / 2 + 1 + 15) & ~15; }

// Index of bin (kx, y, z) in the half spectrum: rows of sp bins (y, z), or
// kx-major planes of (z, y) for k_fft_yz (TR).
template <bool TR>
__device__ __forceinline__ unsigned spec_at(int k, int y, int z, int ny, int nz, int sp) {
    return TR ? ((unsigned)k * (unsigned)nz + (unsigned)z) * (unsigned)ny + (unsigned)y
              : ((unsigned)z * (unsigned)ny + (unsigned)y) * (unsigned)sp + (unsigned)k;
}

// Rows per plane and planes of the x passes.  The two rows of a complex
// sequence are neighbours in memory, 2 j and 2 j + 1 of all ny nz rows, and
// their partner enters both rows' rounding; where ny is odd the pairs run on
// across planes, so there the whole grid counts as one plane (rows, values and
// both forms of the spectrum are contiguous over y and z).
__host__ __device__ int fft_x_rows(int ny, int nz) { return (ny & 1) ? ny * nz : ny; }
__host__ __device__ int fft_x_planes(int ny, int nz) { return (ny & 1) ? 1 : nz; }

// Groups of the x passes: rows y0 .. y0 + 2 pairs - 1 of plane k, in the order
// of memory; a work-group takes I.fxg consecutive ones.
struct XGroup {
    int y0, k;
};
__device__ __forceinline__ XGroup x_group(int lin, int gy, int pairs) {
    const int k = lin / gy;
    return {(lin - k * gy) * 2 * pairs, k};
}

// twiddles of a length into LDS, loads issued XB per thread at a time
template <int NT>
__device__ __forceinline__ void stage_tw(float2 *dst, const float2 *src, int n) {
    constexpr int XB = 4;
    for (int t0 = threadIdx.x; t0 < n; t0 += XB * NT) {
        float2 v[XB];
#pragma unroll
        for (int c = 0; c < XB; ++c) {
            const int t = t0 + c * NT;
            v[c] = t < n ? ld2((const gf2 *)src, t) : make_float2(0.f, 0.f);
        }
#pragma unroll
        for (int c = 0; c < XB; ++c) {
            const int t = t0 + c * NT;
            if (t < n) dst[t] = v[c];
        }
    }
}

// Forward real-to-complex FFT along x into the half spectrum (nx/2 + 1 bins
// per row), fft_x_pairs row pairs of a plane per work-group of FFT_X_THREADS
// threads, I.fxg groups one after the other; XC bounds the complex points
// per group (FFT_X_PTS, or 4 FFT_X_PTS for longer rows), which sizes the
// butterfly registers.  Two real rows a, b travel as one complex row a + i b;
// their spectra are separated with the conjugate symmetry
//   A_k = (Z_k + conj Z_{n-k}) / 2,  B_k = (Z_k - conj Z_{n-k}) / (2 i).
// SRC_F: the rows are those of `in_ext`, or of I.f.  SRC_PSI: they are the
// right side f = Im[psi^* NS(psi)] (the function of k_stencil<MODE_RHS>, the
// same bits), made here from psi, with its neighbours read from the caches,
// instead of by a pass that writes f and one that reads it back.
template <bool P2, int XC, int SRC, bool TR>
__global__ __launch_bounds__(FFT_X_THREADS) void k_fft_fwd(const Inst *__restrict__ insts,
                                                           const int *__restrict__ prefix, int ninst,
                                                           const float *in_ext) {
    extern __shared__ float2 sm[];
    // (kx-major spectrum: neighbouring groups write parts of the same lines,
    // so they run on one XCD)
    const int lbg = TR ? xcd_remap(blockIdx.x, gridDim.x) : (int)blockIdx.x;
    const int ii = find_inst(prefix, ninst, lbg);
    const Inst &I = insts[ii];
    // (the right side from psi is made for even ny only)
    const int nx = I.nx, P = nx / 2 + 1, sp = I.sp;
    const int ny = SRC == SRC_F ? fft_x_rows(I.ny, I.nz) : I.ny, nz = SRC == SRC_F ? fft_x_planes(I.ny, I.nz) : I.nz;
    const int pairs = fft_x_pairs(nx, I.ny);
    const int ss = nx + 1;
    const int gy = (ny + 2 * pairs - 1) / (2 * pairs), ngr = gy * nz;
    const int g0 = (lbg - prefix[ii]) * I.fxg, g1 = min(g0 + I.fxg, ngr);
    float2 *stw = sm + pairs * ss;
    stage_tw<FFT_X_THREADS>(stw, I.twx, nx);
    constexpr bool RHS = SRC != SRC_F, YZ = SRC == SRC_PSI_YZ;
    const gf1 *in = (const gf1 *)(in_ext ? in_ext : I.f);
    const gf2 *__restrict__ psi = RHS ? (const gf2 *)I.psi[I.st->cur] : nullptr;
    gf2 *spec = (gf2 *)I.spec;
    const float inv_nx = 1.0f / (float)nx, inv_p = 1.0f / (float)P, inv_r = 1.0f / (float)(2 * pairs);
    const int tot = pairs * nx;
    const unsigned NXY = (unsigned)nx * (unsigned)ny;
    // PF: a thread holds ML points of every group; those of a real array are
    // loaded for the next plane while the current one is transformed (rows
    // longer than FFT_X_PTS would cost too many registers: they are loaded in
    // batches of ML)
    constexpr bool PF = XC <= FFT_X_PTS;
    constexpr int ML = PF ? XC / FFT_X_THREADS : 4;
    // point t of a group: rows ya = y0 + 2 s and ya + 1, element e
    auto point = [&](int y0, int t, int &s, int &e, bool &va, bool &vb) {
        s = fdiv(t, inv_nx);
        e = t - s * nx;
        const int ya = y0 + 2 * s;
        va = t < tot && ya < ny;
        vb = t < tot && ya + 1 < ny;
    };
    const float cx = I.cx, cy = I.cy, cz = I.cz;
    // f of both rows of a point in plane k (a point without rows computes on
    // row 0 and returns 0)
    auto rhs = [&](XGroup T, int t, float &fa, float &fb) {
        int s, e;
        bool va, vb;
        point(T.y0, t, s, e, va, vb);
        const int k = T.k;
        const int ya = va ? T.y0 + 2 * s : 0, yt = vb ? ya + 1 : ya;
        const int yl = ya == 0 ? ny - 1 : ya - 1, yh = yt == ny - 1 ? 0 : yt + 1;
        const int em = e == 0 ? nx - 1 : e - 1, ep = e == nx - 1 ? 0 : e + 1;
        const bool zm = k > 0, zp = k < nz - 1;
        const unsigned oa = (unsigned)(ya * nx), ob = (unsigned)(yt * nx), m = (unsigned)k * NXY;
        const unsigned mm = zm ? m - NXY : m, mp = zp ? m + NXY : m;
        const float2 ca = ld2(psi, m + oa + e), cb = ld2(psi, m + ob + e);
        const float2 ma = ld2(psi, mm + oa + e), mb = ld2(psi, mm + ob + e);
        const float2 pa = ld2(psi, mp + oa + e), pb = ld2(psi, mp + ob + e);
        const float2 xma = ld2(psi, m + oa + em), xpa = ld2(psi, m + oa + ep);
        const float2 xmb = ld2(psi, m + ob + em), xpb = ld2(psi, m + ob + ep);
        float2 lo = ld2(psi, m + (unsigned)(yl * nx + e)), hi = ld2(psi, m + (unsigned)(yh * nx + e));
        float2 ua = ld2((const gf2 *)I.ux, ya), ub = ld2((const gf2 *)I.ux, yt);
        const float2 wa = ld2((const gf2 *)I.uz, ya), wb = ld2((const gf2 *)I.uz, yt);
        if (ya == 0 || yt == ny - 1) {
            const float2 ph = ld2((const gf2 *)I.P, (unsigned)(k * nx + e));
            if (ya == 0) lo = xcmul(ph, lo);
            if (yt == ny - 1) hi = xcmulc(ph, hi);
        }
        if (YZ) {
            const float2 w = ld2((const gf2 *)I.wz, (unsigned)k);
            ua = xcmul(ua, w);
            ub = xcmul(ub, w);
        }
        fa = va ? rhs_node(ca, nsum(ua, wa, xma, xpa, lo, vb ? cb : hi, ma, pa, zm, zp, cx, cy, cz)) : 0.f;
        fb = vb ? rhs_node(cb, nsum(ub, wb, xmb, xpb, ca, hi, mb, pb, zm, zp, cx, cy, cz)) : 0.f;
    };
    auto load_f = [&](XGroup T, int t, float &fa, float &fb) {
        int s, e;
        bool va, vb;
        point(T.y0, t, s, e, va, vb);
        const size_t o = (size_t)T.k * NXY + (size_t)(T.y0 + 2 * s) * nx + e;
        fa = va ? in[o] : 0.f;
        fb = vb ? in[o + nx] : 0.f;
    };
    auto put = [&](int t, float fa, float fb) {
        if (t < tot) {
            const int s = fdiv(t, inv_nx);
            sm[s * ss + (t - s * nx)] = make_float2(fa, fb);
        }
    };
    float fa[ML], fb[ML];
    if (PF && !RHS) {
#pragma unroll
        for (int c = 0; c < ML; ++c) load_f(x_group(g0, gy, pairs), (int)threadIdx.x + c * FFT_X_THREADS, fa[c], fb[c]);
    }
    for (int g = g0; g < g1; ++g) {
        const XGroup T = x_group(g, gy, pairs);
        const int k = T.k;
        if (RHS) {
#pragma unroll 2
            for (int t = threadIdx.x; t < tot; t += FFT_X_THREADS) {
                float a, b;
                rhs(T, t, a, b);
                put(t, a, b);
            }
        } else if (PF) {
#pragma unroll
            for (int c = 0; c < ML; ++c) put((int)threadIdx.x + c * FFT_X_THREADS, fa[c], fb[c]);
        } else {
            for (int t0 = threadIdx.x; t0 < tot; t0 += ML * FFT_X_THREADS) {
#pragma unroll
                for (int c = 0; c < ML; ++c) load_f(T, t0 + c * FFT_X_THREADS, fa[c], fb[c]);
#pragma unroll
                for (int c = 0; c < ML; ++c) put(t0 + c * FFT_X_THREADS, fa[c], fb[c]);
            }
        }
        __syncthreads();
        if (PF && !RHS && g + 1 < g1) {
#pragma unroll
            for (int c = 0; c < ML; ++c) load_f(x_group(g + 1, gy, pairs), (int)threadIdx.x + c * FFT_X_THREADS, fa[c], fb[c]);
        }
        fft_lds<P2, FFT_X_THREADS, XC>(sm, nx, I.xrad, I.nxrad, pairs, ss, stw, -1.f);
        // TR: consecutive lanes on consecutive rows of one bin
        for (int t = threadIdx.x; t < (TR ? 2 : 1) * pairs * P; t += FFT_X_THREADS) {
            if (TR) {
                const int kx = fdiv(t, inv_r), r = t - kx * 2 * pairs, s = r >> 1;
                const float2 z = sm[s * ss + kx];
                const float2 zc = sm[s * ss + (kx == 0 ? 0 : nx - kx)];
                const float2 v = (r & 1) ? make_float2(0.5f * (z.y + zc.y), -0.5f * (z.x - zc.x))
                                         : make_float2(0.5f * (z.x + zc.x), 0.5f * (z.y - zc.y));
                const int y = T.y0 + r;
                if (y < ny) st2(spec, spec_at<TR>(kx, y, k, ny, nz, sp), v);
            } else {
                const int s = fdiv(t, inv_p), kx = t - s * P;
                const float2 z = sm[s * ss + kx];
                const float2 zc = sm[s * ss + (kx == 0 ? 0 : nx - kx)];
                // A = (z + conj zc)/2, B = (z - conj zc)/(2i)
                const float2 A = make_float2(0.5f * (z.x + zc.x), 0.5f * (z.y - zc.y));
                const float2 B = make_float2(0.5f * (z.y + zc.y), -0.5f * (z.x - zc.x));
                const int ya = T.y0 + 2 * s;
                if (ya < ny) st2(spec, spec_at<TR>(kx, ya, k, ny, nz, sp), A);
                if (ya + 1 < ny) st2(spec, spec_at<TR>(kx, ya + 1, k, ny, nz, sp), B);
            }
        }
        __syncthreads();
    }
}

// The inverse (complex-to-real) along x into mu, with the
// work-group's FP64 partial of the weighted mean of mu (weights: the control
// volumes; the sum of k_mu_mean_partial, which read mu back in a pass of its
// own: 120 us at 1024 x 1024 x 128).
template <bool P2, int XC, bool TR>
__global__ __launch_bounds__(FFT_X_THREADS) void k_fft_inv(const Inst *__restrict__ insts,
                                                           const int *__restrict__ prefix, int ninst) {
    extern __shared__ float2 sm[];
    __shared__ double red[FFT_X_THREADS / 64];
    const int lbg = TR ? xcd_remap(blockIdx.x, gridDim.x) : (int)blockIdx.x;
    const int ii = find_inst(prefix, ninst, lbg);
    const Inst &I = insts[ii];
    const int nx = I.nx, P = nx / 2 + 1, sp = I.sp;
    const int ny = fft_x_rows(I.ny, I.nz), nz = fft_x_planes(I.ny, I.nz);
    const bool flat = ny != I.ny;  // rows of several planes in a group
    const int pairs = fft_x_pairs(nx, I.ny);
    const int ss = nx + 1, R = 2 * pairs;
    const int gy = (ny + R - 1) / R, ngr = gy * nz;
    const int g0 = (lbg - prefix[ii]) * I.fxg, g1 = min(g0 + I.fxg, ngr);
    float2 *stw = sm + pairs * ss;
    stage_tw<FFT_X_THREADS>(stw, I.twx, nx);
    gf1 *out = (gf1 *)I.mu;
    const gf2 *spec = (const gf2 *)I.spec;
    const gf1 *volz = (const gf1 *)I.lev[0].vol[2];
    const float inv_nx = 1.0f / (float)nx, inv_r = 1.0f / (float)R;
    const int tot = pairs * nx;
    const unsigned NXY = (unsigned)nx * (unsigned)ny;
    constexpr bool PF = XC <= FFT_X_PTS;
    constexpr int ML = PF ? XC / FFT_X_THREADS : 4;
    // W = A + i B of bin k <= nx/2 of a pair's rows, and of bin nx - k by
    // symmetry.  TR: one row's value per load (A or B), consecutive lanes on
    // consecutive rows; otherwise both rows' values of a bin.
    constexpr int NV = TR ? 1 : 2;
    const int items = TR ? R * P : tot;  // loads of a group
    constexpr int MV = TR ? (XC + 64 + FFT_X_THREADS - 1) / FFT_X_THREADS : ML;  // R P <= pairs (nx + 2)
    float2 v[PF ? MV : 4][NV];
    auto load = [&](XGroup T, int t, float2 *w) {
        const int z = T.k;
        if (TR) {
            const int kx = fdiv(t, inv_r), r = t - kx * R, y = T.y0 + r;
            w[0] = (t < items && y < ny) ? ld2(spec, spec_at<TR>(kx, y, z, ny, nz, sp)) : make_float2(0.f, 0.f);
        } else {
            const int s = fdiv(t, inv_nx), k = t - s * nx, kk = k < P ? k : nx - k, ya = T.y0 + 2 * s;
            w[0] = (t < items && ya < ny) ? ld2(spec, spec_at<TR>(kk, ya, z, ny, nz, sp)) : make_float2(0.f, 0.f);
            w[NV - 1] = (t < items && ya + 1 < ny) ? ld2(spec, spec_at<TR>(kk, ya + 1, z, ny, nz, sp))
                                                   : make_float2(0.f, 0.f);
        }
    };
    auto put = [&](int t, const float2 *w) {
        if (t >= items) return;
        if (TR) {
            // rows a and b of a pair sit in neighbouring lanes: lane a makes
            // W_k = A + i B, lane b W_{n-k} = conj A + i conj B
            const int kx = fdiv(t, inv_r), r = t - kx * R, s = r >> 1;
            const float2 o = make_float2(__shfl_xor(w[0].x, 1, 64), __shfl_xor(w[0].y, 1, 64));
            if (!(r & 1)) sm[s * ss + kx] = make_float2(w[0].x - o.y, w[0].y + o.x);
            else if (kx > 0 && kx < nx - kx) sm[s * ss + nx - kx] = make_float2(o.x + w[0].y, -o.y + w[0].x);
        } else {
            const int s = fdiv(t, inv_nx), k = t - s * nx;
            float2 a = w[0], b = w[NV - 1];
            if (k >= P) { a.y = -a.y; b.y = -b.y; }
            sm[s * ss + k] = make_float2(a.x - b.y, a.y + b.x);
        }
    };
    constexpr int NB = PF ? MV : 4;
    if (PF) {
#pragma unroll
        for (int c = 0; c < NB; ++c) load(x_group(g0, gy, pairs), (int)threadIdx.x + c * FFT_X_THREADS, v[c]);
    }
    double acc = 0.0;
    for (int g = g0; g < g1; ++g) {
        const XGroup T = x_group(g, gy, pairs);
        const int k = T.k;
        if (PF) {
#pragma unroll
            for (int c = 0; c < NB; ++c) put((int)threadIdx.x + c * FFT_X_THREADS, v[c]);
        } else {
            for (int t0 = threadIdx.x; t0 < items; t0 += NB * FFT_X_THREADS) {
#pragma unroll
                for (int c = 0; c < NB; ++c) load(T, t0 + c * FFT_X_THREADS, v[c]);
#pragma unroll
                for (int c = 0; c < NB; ++c) put(t0 + c * FFT_X_THREADS, v[c]);
            }
        }
        __syncthreads();
        if (PF && g + 1 < g1) {
#pragma unroll
            for (int c = 0; c < NB; ++c) load(x_group(g + 1, gy, pairs), (int)threadIdx.x + c * FFT_X_THREADS, v[c]);
        }
        fft_lds<P2, FFT_X_THREADS, XC>(sm, nx, I.xrad, I.nxrad, pairs, ss, stw, +1.f);
        double sum = 0.0;
        for (int t = threadIdx.x; t < tot; t += FFT_X_THREADS) {
            const int s = fdiv(t, inv_nx), e = t - s * nx;
            const int ya = T.y0 + 2 * s;
            const float2 w = sm[s * ss + e];
            const unsigned m = (unsigned)k * NXY + (unsigned)(ya * nx + e);
            if (ya < ny) {
                out[m] = w.x;
                sum += flat ? (double)volz[ya / I.ny] * (double)w.x : (double)w.x;
            }
            if (ya + 1 < ny) {
                out[m + nx] = w.y;
                sum += flat ? (double)volz[(ya + 1) / I.ny] * (double)w.y : (double)w.y;
            }
        }
        acc += flat ? sum : (double)volz[k] * sum;
        __syncthreads();
    }
    // x and y are periodic: one control volume each
    const double vxy = (double)I.lev[0].vol[0][0] * I.lev[0].vol[1][0];
    const double s = wg_sum<FFT_X_THREADS>(acc * vxy, red);
    if (threadIdx.x == 0) I.part[lbg - prefix[ii]] = s;
}

// FFT along y of the half spectrum, forward (dir = -1) or inverse (+1):
// a work-group takes one tile of fft_y_plan -- TK consecutive kx of one
// plane on tall grids, G whole planes on short ones -- all y.  Consecutive
// tiles share 128-byte lines, so neighbouring logical tiles run on one XCD.
// (P2: 64 registers, so that two work-groups share a CU; with 66 the pass
// took 534 us at 1024 x 1024 x 128 instead of 320)
template <bool P2>
__global__ __launch_bounds__(FFT_THREADS, P2 ? 8 : 4) void k_fft_y(const Inst *__restrict__ insts,
                                                       const int *__restrict__ prefix, int ninst,
                                                       int dir) {
    extern __shared__ float2 sm[];
    const int ii = find_inst(prefix, ninst, blockIdx.x);
    const Inst &I = insts[ii];
    const int nx = I.nx, ny = I.ny, nz = I.nz, P = nx / 2 + 1, sp = I.sp;
    const FftYPlan pl = fft_y_plan(nx, ny, nz);
    const int TK = pl.TK;
    const int nblk = prefix[ii + 1] - prefix[ii];
    const int lb = xcd_remap(blockIdx.x - prefix[ii], nblk);
    const int zt = lb / pl.ntk, j = lb - zt * pl.ntk;
    // the tile starts at kx = r0 of plane z0; column c is kx = r0 + c of
    // that plane (per-plane tiles) or kx = c - q P of plane z0 + q, q =
    // floor(c / P) (whole planes, r0 = 0); offsets within a tile fit 32 bits
    const int z0 = zt * pl.G, r0 = j * TK;
    const bool whole = pl.ntk == 1;
    const int tk = whole ? min(pl.G, nz - z0) * P : min(TK, P - r0);
    const unsigned zs = (unsigned)ny * (unsigned)sp;
    const gf2 *__restrict__ specr = (const gf2 *)(I.spec + (size_t)z0 * zs);
    gf2 *__restrict__ specw = (gf2 *)(I.spec + (size_t)z0 * zs);
    const float inv_tk = 1.0f / (float)TK, inv_p = 1.0f / (float)P;
    auto col = [&](int c) -> unsigned {
        if (!whole) return (unsigned)(r0 + c);
        const int q = fdiv(c, inv_p);
        return (unsigned)q * zs + (unsigned)(c - q * P);
    };
    // columns sit ss = ny + 1 apart in LDS: the staging loop writes (and the
    // final loop reads) TK columns per y with consecutive lanes, which a
    // power-of-two stride would put on one bank
    const int ss = fft_y_stride(ny);
    float2 *stw = sm + TK * ss;
    for (int t = threadIdx.x; t < ny; t += FFT_THREADS) stw[t] = ld2((const gf2 *)I.twy, t);
    // loads are issued YB per thread at a time before any of them is
    // stored to LDS
    constexpr int YB = 8;
    const int tot = ny * TK;
    for (int t0 = threadIdx.x; t0 < tot; t0 += YB * FFT_THREADS) {
        float2 v[YB];
#pragma unroll
        for (int q = 0; q < YB; ++q) {
            const int t = t0 + q * FFT_THREADS;
            const int y = fdiv(t, inv_tk), c = t - y * TK;
            v[q] = (t < tot && c < tk) ? ld2(specr, col(c) + (unsigned)(y * sp)) : make_float2(0.f, 0.f);
        }
#pragma unroll
        for (int q = 0; q < YB; ++q) {
            const int t = t0 + q * FFT_THREADS;
            const int y = fdiv(t, inv_tk), c = t - y * TK;
            if (t < tot) sm[c * ss + y] = v[q];
        }
    }
    __syncthreads();
    fft_lds<P2, FFT_THREADS, FFT_MAXPTS>(sm, ny, I.yrad, I.nyrad, TK, ss, stw, (float)dir);
    for (int t = threadIdx.x; t < ny * TK; t += FFT_THREADS) {
        const int y = fdiv(t, inv_tk), c = t - y * TK;
        if (c < tk) st2(specw, col(c) + (unsigned)(y * sp), sm[c * ss + y]);
    }
}

// Set-up of the spectral solver of instance `inst`: twiddle tables
// exp(-2 pi i k / n) for x and y (FP64 arguments, rounded once to FP32), and
// for every z system its Thomas pivots ip_k = 1 / (b_k - a_k c'_{k-1}),
// c'_k = c_k ip_k, in FP64, stored column by column at ((ky P + kx) nz + k).
// The operator does not change between steps, so this runs once.
__global__ void k_fft_tables(const Inst *__restrict__ insts, int inst) {
    const Inst &I = insts[inst];
    const int nx = I.nx, ny = I.ny, nz = I.nz, P = nx / 2 + 1;
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < nx) {
        double s, c;
        sincospi(-2.0 * (double)t / (double)nx, &s, &c);
        I.twx[t] = make_float2((float)c, (float)s);
    }
    if (t < ny) {
        double s, c;
        sincospi(-2.0 * (double)t / (double)ny, &s, &c);
        I.twy[t] = make_float2((float)c, (float)s);
    }
    if (t < ny * P) {
        const int ky = t / P, kx = t - ky * P;
        const double cz = I.cz, cx = I.cx, cy = I.cy;
        const double lam = cx * (2.0 - 2.0 * cospi(2.0 * kx / (double)nx)) +
                           cy * (2.0 - 2.0 * cospi(2.0 * ky / (double)ny));
        const bool singular = (kx == 0 && ky == 0);
        double cprev = 0.0;
        double *ip = I.zip + (size_t)t * nz;
        for (int k = 0; k < nz; ++k) {
            double a, c;
            zrow(k, nz, cz, singular, a, c);
            double b = (nz == 1) ? -lam : -(lam + 2.0 * cz);
            if (singular && k == 0) b = 1.0;
            const double p = 1.0 / (b - a * cprev);
            ip[k] = p;
            cprev = c * p;
        }
    }
}

#define TDGL_FFT_X(P2, XC, TR)                                                                        \
    template __global__ void k_fft_fwd<P2, XC, SRC_F, TR>(const Inst *, const int *, int, const float *); \
    template __global__ void k_fft_inv<P2, XC, TR>(const Inst *, const int *, int);
#define TDGL_FFT_XP(P2)                                                                                          \
    template __global__ void k_fft_fwd<P2, FFT_X_PTS, SRC_PSI, true>(const Inst *, const int *, int, const float *); \
    template __global__ void k_fft_fwd<P2, FFT_X_PTS, SRC_PSI_YZ, true>(const Inst *, const int *, int, const float *);
TDGL_FFT_X(false, FFT_X_PTS, false)
TDGL_FFT_X(true, FFT_X_PTS, false)
TDGL_FFT_X(false, FFT_X_PTS, true)
TDGL_FFT_X(true, FFT_X_PTS, true)
TDGL_FFT_X(false, 4 * FFT_X_PTS, false)
TDGL_FFT_X(true, 4 * FFT_X_PTS, false)
TDGL_FFT_XP(false)
TDGL_FFT_XP(true)
#undef TDGL_FFT_XP
#undef TDGL_FFT_X
template __global__ void k_fft_y<false>(const Inst *, const int *, int, int);
template __global__ void k_fft_y<true>(const Inst *, const int *, int, int);

// The z systems, one per (kx, ky), in double precision.  A work-group loads
// a tile of ZTK consecutive kx at one ky and all z (coalesced rows); each
// wavefront then solves the columns of the tile, one or two at a time.
// With the pivots of the set-up, Thomas' two sweeps are first-order linear
// recurrences,
//   y_k = -a_k ip_k y_{k-1} + ip_k d_k,   mu_k = -c_k ip_k mu_{k+1} + y_k,
// i.e. compositions of affine maps, which a segment of L lanes evaluates as
// a prefix scan (lane l owns rows l RPL .. l RPL + RPL - 1): compose the
// lane's maps, scan the lane maps across the segment with shuffles, then
// replay the rows from the lane's incoming value.  The result is scaled by
// 1/(nx ny) (the two inverse FFTs are unnormalised).
constexpr int ZTK = FFT_ZTK;
constexpr int ZPAD = ZTK + 1;  // LDS row stride (float2): spreads the column reads over banks
__host__ __device__ size_t fft_z_lds(int nz) { return (size_t)nz * ZPAD * sizeof(float2); }

// Thin boxes (nz <= FFT_ZSERIAL, e.g. a film of one plane): the cost of the
// scan is per system, not per row, so here one lane takes one (kx, ky)
// system, with consecutive lanes on consecutive kx (coalesced rows), and runs
// Thomas' two sweeps with the stored pivots in registers.
__device__ __forceinline__ void zsolve_lane(const Inst &I, int lb) {
    const int nx = I.nx, ny = I.ny, nz = I.nz, P = nx / 2 + 1;
    const int col = lb * ZS_THREADS + threadIdx.x;
    if (col >= ny * P) return;
    const int ky = col / P, kx = col - ky * P;
    const size_t zstride = (size_t)ny * I.sp;
    float2 *spec = I.spec + (size_t)ky * I.sp + kx;
    const double *ipc = I.zip + (size_t)col * nz;
    const double cz = I.cz;
    const double scale = 1.0 / ((double)nx * (double)ny);
    const bool singular = (kx == 0 && ky == 0);
    double yr[FFT_ZSERIAL], yi[FFT_ZSERIAL];
#pragma unroll
    for (int k = 0; k < FFT_ZSERIAL; ++k) {
        const float2 v = k < nz ? spec[(size_t)k * zstride] : make_float2(0.f, 0.f);
        yr[k] = v.x;
        yi[k] = v.y;
    }
    // weighted mean over z (1/2 on the two end rows of an open axis)
    auto wmean = [&](double &mr, double &mi) {
        double sr = 0.0, si = 0.0, sw = 0.0;
#pragma unroll
        for (int k = 0; k < FFT_ZSERIAL; ++k)
            if (k < nz) {
                const double wk = (nz > 1 && (k == 0 || k == nz - 1)) ? 0.5 : 1.0;
                sr += wk * yr[k];
                si += wk * yi[k];
                sw += wk;
            }
        mr = sr / sw;
        mi = si / sw;
    };
    if (singular) {
        // project the right side onto the range and pin row 0
        double mr, mi;
        wmean(mr, mi);
#pragma unroll
        for (int k = 0; k < FFT_ZSERIAL; ++k) {
            yr[k] -= mr;
            yi[k] -= mi;
        }
        yr[0] = 0.0;
        yi[0] = 0.0;
    }
    double ur = 0.0, ui = 0.0;
#pragma unroll
    for (int k = 0; k < FFT_ZSERIAL; ++k)
        if (k < nz) {
            double a, cc;
            zrow(k, nz, cz, singular, a, cc);
            const double ip = ipc[k];
            const double Ak = -a * ip, s = ip * scale;
            ur = Ak * ur + s * yr[k];
            ui = Ak * ui + s * yi[k];
            yr[k] = ur;
            yi[k] = ui;
        }
    double xr = 0.0, xi = 0.0;
#pragma unroll
    for (int k = FFT_ZSERIAL - 1; k >= 0; --k)
        if (k < nz) {
            double a, cc;
            zrow(k, nz, cz, singular, a, cc);
            const double Ck = -cc * ipc[k];
            xr = Ck * xr + yr[k];
            xi = Ck * xi + yi[k];
            yr[k] = xr;
            yi[k] = xi;
        }
    if (singular) {
        // shift the constant mode to zero weighted mean
        double mr, mi;
        wmean(mr, mi);
#pragma unroll
        for (int k = 0; k < FFT_ZSERIAL; ++k) {
            yr[k] -= mr;
            yi[k] -= mi;
        }
    }
#pragma unroll
    for (int k = 0; k < FFT_ZSERIAL; ++k)
        if (k < nz) spec[(size_t)k * zstride] = make_float2((float)yr[k], (float)yi[k]);
}

// RMAX: z rows per lane of the scan for every instance of the launch (2 up
// to nz = 64, else 4): fewer registers, more work-groups per CU for the
// shallow boxes.  Columns of up to 32 RMAX rows are scanned on 32-lane
// segments (two columns per wavefront), deeper ones on the whole
// wavefront.
template <int RMAX>
__global__ __launch_bounds__(ZS_THREADS) void k_fft_zsolve(const Inst *__restrict__ insts,
                                                            const int *__restrict__ prefix,
                                                            int ninst) {
    extern __shared__ float2 tile[];
    const int ii = find_inst(prefix, ninst, blockIdx.x);
    const Inst &I = insts[ii];
    if (I.nz <= FFT_ZSERIAL) {
        zsolve_lane(I, blockIdx.x - prefix[ii]);
        return;
    }
    const int nx = I.nx, ny = I.ny, nz = I.nz, P = nx / 2 + 1, sp = I.sp;
    const int ntk = (P + ZTK - 1) / ZTK;
    const int lb = blockIdx.x - prefix[ii];
    const int ky = lb / ntk, kx0 = (lb - ky * ntk) * ZTK;
    const int tk = min(ZTK, P - kx0);
    const unsigned zstride = (unsigned)ny * (unsigned)sp;
    gf2 *spec = (gf2 *)(I.spec + (size_t)ky * sp + kx0);
    // loads are issued ZB per thread at a time before any of them is
    // stored to LDS
    constexpr int ZB = 8;
    const int tot = nz * ZTK;
    for (int t0 = threadIdx.x; t0 < tot; t0 += ZB * ZS_THREADS) {
        float2 v[ZB];
#pragma unroll
        for (int q = 0; q < ZB; ++q) {
            const int t = t0 + q * ZS_THREADS;
            const int k = t / ZTK, c = t - k * ZTK;
            v[q] = (t < tot && c < tk) ? ld2(spec, (unsigned)k * zstride + c) : make_float2(0.f, 0.f);
        }
#pragma unroll
        for (int q = 0; q < ZB; ++q) {
            const int t = t0 + q * ZS_THREADS;
            const int k = t / ZTK, c = t - k * ZTK;
            if (t < tot) tile[k * ZPAD + c] = v[q];
        }
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const double cz = I.cz;
    const double scale = 1.0 / ((double)nx * (double)ny);
    static_assert(RMAX * 64 <= FFT_ZMAX, "scan rows per lane");
    // the scan runs on segments of L lanes, 64 / L columns per wavefront at
    // a time: the scan's cost is per column, so columns of up to 32 RMAX
    // rows take 32-lane segments (with nz <= 32 the same maps are composed
    // in the same order as on 64 lanes, whose upper half would only hold
    // identity maps)
    const int L = nz <= 32 * RMAX ? 32 : 64;
    const int S = 64 / L;
    const int sl = lane & (L - 1), sg = lane / L;
    const int rpl = (nz + L - 1) / L;
    const int k0 = sl * rpl;
    // pivots of the wavefront's next column are loaded while the current
    // one is solved
    double ipn[RMAX];
    auto load_piv = [&](int c, double *dst) {
        const gd1 *ipc = (const gd1 *)(I.zip + ((size_t)ky * P + kx0 + c) * nz);
#pragma unroll
        for (int q = 0; q < RMAX; ++q) {
            const int k = k0 + q;
            dst[q] = (c < tk && q < rpl && k < nz) ? ipc[k] : 0.0;
        }
    };
    load_piv(w * S + sg, ipn);
    for (int c = w * S + sg; c < tk; c += 4 * S) {
        const int kx = kx0 + c;
        const bool singular = (kx == 0 && ky == 0);
        double yr[RMAX], yi[RMAX], ip[RMAX];
#pragma unroll
        for (int q = 0; q < RMAX; ++q) ip[q] = ipn[q];
        load_piv(c + 4 * S, ipn);
#pragma unroll
        for (int q = 0; q < RMAX; ++q) {
            const int k = k0 + q;
            const bool ok = q < rpl && k < nz;
            const float2 v = ok ? tile[k * ZPAD + c] : make_float2(0.f, 0.f);
            yr[q] = v.x;
            yi[q] = v.y;
        }
        // the singular column: project the right side onto the range
        // (zero weighted mean) and pin row 0
        if (singular) {
            double sr = 0.0, si = 0.0, sw = 0.0;
#pragma unroll
            for (int q = 0; q < RMAX; ++q) {
                const int k = k0 + q;
                if (q < rpl && k < nz) {
                    const double wk = (nz > 1 && (k == 0 || k == nz - 1)) ? 0.5 : 1.0;
                    sr += wk * yr[q];
                    si += wk * yi[q];
                    sw += wk;
                }
            }
            for (int o = L / 2; o > 0; o >>= 1) {
                sr += __shfl_xor(sr, o, L);
                si += __shfl_xor(si, o, L);
                sw += __shfl_xor(sw, o, L);
            }
#pragma unroll
            for (int q = 0; q < RMAX; ++q) {
                yr[q] -= sr / sw;
                yi[q] -= si / sw;
                if (k0 + q == 0) { yr[q] = 0.0; yi[q] = 0.0; }
            }
        }
        // forward sweep: lane map y_out = A y_in + B
        double A = 1.0, Br = 0.0, Bi = 0.0;
#pragma unroll
        for (int q = 0; q < RMAX; ++q) {
            const int k = k0 + q;
            if (q < rpl && k < nz) {
                double a, cc;
                zrow(k, nz, cz, singular, a, cc);
                const double Ak = -a * ip[q], s = ip[q] * scale;
                Br = Ak * Br + s * yr[q];
                Bi = Ak * Bi + s * yi[q];
                A = Ak * A;
            }
        }
        for (int o = 1; o < L; o <<= 1) {
            const double pA = __shfl_up(A, o, L), pr = __shfl_up(Br, o, L), pi = __shfl_up(Bi, o, L);
            if (sl >= o) {
                Br = A * pr + Br;
                Bi = A * pi + Bi;
                A = A * pA;
            }
        }
        double ur = __shfl_up(Br, 1, L), ui = __shfl_up(Bi, 1, L);
        if (sl == 0) { ur = 0.0; ui = 0.0; }
#pragma unroll
        for (int q = 0; q < RMAX; ++q) {
            const int k = k0 + q;
            if (q < rpl && k < nz) {
                double a, cc;
                zrow(k, nz, cz, singular, a, cc);
                const double Ak = -a * ip[q], s = ip[q] * scale;
                ur = Ak * ur + s * yr[q];
                ui = Ak * ui + s * yi[q];
                yr[q] = ur;
                yi[q] = ui;
            }
        }
        // backward sweep: lane map x_first = C x_in + D, x_in = mu of the
        // next lane's first row
        double C = 1.0, Dr = 0.0, Di = 0.0;
#pragma unroll
        for (int q = RMAX - 1; q >= 0; --q) {
            const int k = k0 + q;
            if (q < rpl && k < nz) {
                double a, cc;
                zrow(k, nz, cz, singular, a, cc);
                const double Ck = -cc * ip[q];
                Dr = Ck * Dr + yr[q];
                Di = Ck * Di + yi[q];
                C = Ck * C;
            }
        }
        for (int o = 1; o < L; o <<= 1) {
            const double nC = __shfl_down(C, o, L), nr = __shfl_down(Dr, o, L), ni = __shfl_down(Di, o, L);
            if (sl + o < L) {
                Dr = C * nr + Dr;
                Di = C * ni + Di;
                C = C * nC;
            }
        }
        double xr = __shfl_down(Dr, 1, L), xi = __shfl_down(Di, 1, L);
        if (sl == L - 1) { xr = 0.0; xi = 0.0; }
#pragma unroll
        for (int q = RMAX - 1; q >= 0; --q) {
            const int k = k0 + q;
            if (q < rpl && k < nz) {
                double a, cc;
                zrow(k, nz, cz, singular, a, cc);
                const double Ck = -cc * ip[q];
                xr = Ck * xr + yr[q];
                xi = Ck * xi + yi[q];
                yr[q] = xr;
                yi[q] = xi;
            }
        }
        if (singular) {
            // shift the constant mode to zero weighted mean
            double sr = 0.0, si = 0.0, sw = 0.0;
#pragma unroll
            for (int q = 0; q < RMAX; ++q) {
                const int k = k0 + q;
                if (q < rpl && k < nz) {
                    const double wk = (nz > 1 && (k == 0 || k == nz - 1)) ? 0.5 : 1.0;
                    sr += wk * yr[q];
                    si += wk * yi[q];
                    sw += wk;
                }
            }
            for (int o = L / 2; o > 0; o >>= 1) {
                sr += __shfl_xor(sr, o, L);
                si += __shfl_xor(si, o, L);
                sw += __shfl_xor(sw, o, L);
            }
#pragma unroll
            for (int q = 0; q < RMAX; ++q) {
                yr[q] -= sr / sw;
                yi[q] -= si / sw;
            }
        }
#pragma unroll
        for (int q = 0; q < RMAX; ++q) {
            const int k = k0 + q;
            if (q < rpl && k < nz) tile[k * ZPAD + c] = make_float2((float)yr[q], (float)yi[q]);
        }
    }
    __syncthreads();
    for (int t = threadIdx.x; t < nz * ZTK; t += ZS_THREADS) {
        const int k = t / ZTK, c = t - k * ZTK;
        if (c < tk) st2(spec, (unsigned)k * zstride + c, tile[k * ZPAD + c]);
    }
}

// The y transforms and the z systems of I.fyz kx planes (kx-major half
// spectrum, all y and z of a plane contiguous) in one work-group: forward FFT
// along y, Thomas' sweeps along z, inverse FFT, in LDS, so the spectrum is
// read and written once and in whole lines instead of three times.  64 x 64 x
// 64: 10.6 + 7.0 + 10.6 us as three kernels.  The z systems are the scans of
// k_fft_zsolve on short segments: YZ_RPL rows per lane and the fewest lanes
// that hold a system (16 up to 64 planes).
constexpr int YZ_THREADS = FFT_YZ_THREADS, YZ_RPL = 4;
// The value of the lane O below (above) within a row of 16 lanes, by DPP
// moves: a double through __shfl costs two LDS permutes.  Lanes without one
// get their own.
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
    const long long b = __double_as_longlong(v);
    const int lo = (int)b, hi = (int)(b >> 32);
    const unsigned l2 = (unsigned)__builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, false);
    const unsigned h2 = (unsigned)__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, false);
    return __longlong_as_double((long long)(((unsigned long long)h2 << 32) | l2));
}
template <int O>
__device__ __forceinline__ double lane_up(double v) { return dpp_move<0x110 + O>(v); }    // row_shr
template <int O>
__device__ __forceinline__ double lane_down(double v) { return dpp_move<0x100 + O>(v); }  // row_shl

template <bool P2>
__global__ __launch_bounds__(YZ_THREADS) void k_fft_yz(const Inst *__restrict__ insts,
                                                       const int *__restrict__ prefix, int ninst) {
    extern __shared__ float2 sm[];
    const int ii = find_inst(prefix, ninst, blockIdx.x);
    const Inst &I = insts[ii];
    const int nx = I.nx, ny = I.ny, nz = I.nz, P = nx / 2 + 1;
    const int G = I.fyz, kx0 = (blockIdx.x - prefix[ii]) * G, g = min(G, P - kx0);
    const int ss = ny + 1, nseq = g * nz, tot = nseq * ny;
    float2 *stw = sm + G * nz * ss;
    stage_tw<YZ_THREADS>(stw, I.twy, ny);
    gf2 *spec = (gf2 *)I.spec + (size_t)kx0 * nz * ny;
    const float inv_ny = 1.0f / (float)ny;
    constexpr int YB = 8;
    for (int t0 = threadIdx.x; t0 < tot; t0 += YB * YZ_THREADS) {
        float2 v[YB];
#pragma unroll
        for (int q = 0; q < YB; ++q) {
            const int t = t0 + q * YZ_THREADS;
            v[q] = t < tot ? ld2(spec, t) : make_float2(0.f, 0.f);
        }
#pragma unroll
        for (int q = 0; q < YB; ++q) {
            const int t = t0 + q * YZ_THREADS;
            const int s = fdiv(t, inv_ny);
            if (t < tot) sm[s * ss + (t - s * ny)] = v[q];
        }
    }
    __syncthreads();
    fft_lds_batches<P2>(sm, ny, I.yrad, I.nyrad, nseq, ss, stw, -1.f);
    // column c of the group: ky = c mod ny of kx plane c / ny.  Real and
    // imaginary parts are systems of their own (the matrix is real): a segment
    // of L lanes solves one part, lane sl holds rows sl YZ_RPL .. + YZ_RPL - 1.
    // Rows past nz are identity maps.
    int L = 1;
    while (L * YZ_RPL < nz) L <<= 1;
    const int sl = (int)threadIdx.x & (L - 1), k0 = sl * YZ_RPL;
    const double cz = I.cz;
    const double scale = 1.0 / ((double)nx * (double)ny);
    const int per = YZ_THREADS / L;  // parts at a time
    const int npart = 2 * g * ny;
    for (int c0 = 0; c0 < npart; c0 += per) {
        const int cp = c0 + (int)threadIdx.x / L;
        const bool on = cp < npart;
        const int c = on ? cp >> 1 : 0;
        const int pl = fdiv(c, inv_ny), ky = c - pl * ny, kx = kx0 + pl;
        const bool singular = kx == 0 && ky == 0;
        const gd1 *ipc = (const gd1 *)(I.zip + ((size_t)ky * P + kx) * nz);
        float *col = (float *)(sm + pl * nz * ss + ky) + (cp & 1);
        double y[YZ_RPL], ip[YZ_RPL];
#pragma unroll
        for (int q = 0; q < YZ_RPL; ++q) ip[q] = ipc[min(k0 + q, nz - 1)];
#pragma unroll
        for (int q = 0; q < YZ_RPL; ++q) y[q] = (double)col[2 * min(k0 + q, nz - 1) * ss];
        // weighted mean over z of the segment's system
        auto wmean = [&]() {
            double s = 0.0, sw = 0.0;
#pragma unroll
            for (int q = 0; q < YZ_RPL; ++q) {
                const int k = k0 + q;
                const double wk = k < nz ? ((nz > 1 && (k == 0 || k == nz - 1)) ? 0.5 : 1.0) : 0.0;
                s += wk * y[q];
                sw += wk;
            }
            for (int o = L / 2; o > 0; o >>= 1) {
                s += __shfl_xor(s, o, L);
                sw += __shfl_xor(sw, o, L);
            }
            return s / sw;
        };
        // the constant mode (among the first systems of the instance's first
        // work-group): projected onto the range, row 0 pinned
        const bool has0 = kx0 == 0 && c0 == 0;
        if (has0) {
            const double m = wmean();
            if (singular) {
#pragma unroll
                for (int q = 0; q < YZ_RPL; ++q) y[q] -= m;
                if (k0 == 0) y[0] = 0.0;
            }
        }
        // row k's maps: forward y_k = Af y_{k-1} + s y, backward x_k = Ab
        // x_{k+1} + y_k
        auto fwd = [&](int q, double &s) {
            const int k = k0 + q;
            double a, cu;
            zrow(k, nz, cz, singular, a, cu);
            s = k < nz ? ip[q] * scale : 0.0;
            return k < nz ? -a * ip[q] : 1.0;
        };
        auto bwd = [&](int q) {
            const int k = k0 + q;
            double a, cu;
            zrow(k, nz, cz, singular, a, cu);
            return k < nz ? -cu * ip[q] : 1.0;
        };
        // forward sweep: the lane's map y_out = A y_in + B, scanned over the
        // segment, then the rows from the lane's incoming value
        double A = 1.0, B = 0.0;
#pragma unroll
        for (int q = 0; q < YZ_RPL; ++q) {
            double s;
            const double Ak = fwd(q, s);
            B = Ak * B + s * y[q];
            A = Ak * A;
        }
        auto fstep = [&](double pA, double pB, int o) {
            if (sl >= o) {
                B = A * pB + B;
                A = A * pA;
            }
        };
        // (segments beyond a DPP row of 16 lanes shuffle through LDS)
        if (L <= 16) {
            if (L > 1) fstep(lane_up<1>(A), lane_up<1>(B), 1);
            if (L > 2) fstep(lane_up<2>(A), lane_up<2>(B), 2);
            if (L > 4) fstep(lane_up<4>(A), lane_up<4>(B), 4);
            if (L > 8) fstep(lane_up<8>(A), lane_up<8>(B), 8);
        } else {
            for (int o = 1; o < L; o <<= 1) fstep(__shfl_up(A, o, 64), __shfl_up(B, o, 64), o);
        }
        double u = L <= 16 ? lane_up<1>(B) : __shfl_up(B, 1, 64);
        if (sl == 0) u = 0.0;
#pragma unroll
        for (int q = 0; q < YZ_RPL; ++q) {
            double s;
            const double Ak = fwd(q, s);
            u = Ak * u + s * y[q];
            y[q] = k0 + q < nz ? u : 0.0;
        }
        // backward sweep: x_first = A x_in + B, x_in the next lane's first row
        A = 1.0;
        B = 0.0;
#pragma unroll
        for (int q = YZ_RPL - 1; q >= 0; --q) {
            const double Ck = bwd(q);
            B = Ck * B + y[q];
            A = Ck * A;
        }
        auto bstep = [&](double nA, double nB, int o) {
            if (sl + o < L) {
                B = A * nB + B;
                A = A * nA;
            }
        };
        if (L <= 16) {
            if (L > 1) bstep(lane_down<1>(A), lane_down<1>(B), 1);
            if (L > 2) bstep(lane_down<2>(A), lane_down<2>(B), 2);
            if (L > 4) bstep(lane_down<4>(A), lane_down<4>(B), 4);
            if (L > 8) bstep(lane_down<8>(A), lane_down<8>(B), 8);
        } else {
            for (int o = 1; o < L; o <<= 1) bstep(__shfl_down(A, o, 64), __shfl_down(B, o, 64), o);
        }
        double x = L <= 16 ? lane_down<1>(B) : __shfl_down(B, 1, 64);
        if (sl == L - 1) x = 0.0;
#pragma unroll
        for (int q = YZ_RPL - 1; q >= 0; --q) {
            x = bwd(q) * x + y[q];
            y[q] = x;
        }
        if (has0) {
            // the constant mode shifted to zero weighted mean
            const double m = wmean();
            if (singular) {
#pragma unroll
                for (int q = 0; q < YZ_RPL; ++q) y[q] -= m;
            }
        }
        if (on) {
#pragma unroll
            for (int q = 0; q < YZ_RPL; ++q) {
                const int k = k0 + q;
                if (k < nz) col[2 * k * ss] = (float)y[q];
            }
        }
    }
    __syncthreads();
    fft_lds_batches<P2>(sm, ny, I.yrad, I.nyrad, nseq, ss, stw, +1.f);
    for (int t = threadIdx.x; t < tot; t += YZ_THREADS) {
        const int s = fdiv(t, inv_ny);
        st2(spec, t, sm[s * ss + (t - s * ny)]);
    }
}
template __global__ void k_fft_yz<false>(const Inst *, const int *, int);
template __global__ void k_fft_yz<true>(const Inst *, const int *, int);

template __global__ void k_fft_zsolve<2>(const Inst *, const int *, int);
template __global__ void k_fft_zsolve<4>(const Inst *, const int *, int);

}  // namespace tdgl
