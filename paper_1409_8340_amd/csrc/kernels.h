// kernels.h -- declarations of the libtdgl kernels (defined in k_*.hip).
#pragma once
#include "tdgl_dev.h"

namespace tdgl {

enum { MODE_FIRST = 0, MODE_SWEEP = 1, MODE_RHS = 2, MODE_ENERGY = 3, MODE_FIRSTN = 4 };
// MODE_FIRSTN: MODE_FIRST with the Langevin term (a separate instantiation,
// so that the noiseless assemble carries none of the generator's registers).
constexpr bool is_first_mode(int m) { return m == MODE_FIRST || m == MODE_FIRSTN; }
constexpr int JAV_CPT = 16;     // least cells per thread of the flat reductions (a multiple of 8)
constexpr int JAV_CPT_MAX = 64; // most cells per thread, taken while 2048 or more work-groups remain
constexpr int CO_THREADS = 1024;
// Most nodes of the levels that k_mg_tail takes, 12 bytes of LDS each: one CU's
// work per level against launches of 5 us.  Whole runs of 192 x 101 x 33 with
// the tail at 12 x 8 x 3 alone / from 24 x 14 x 5 (1968 nodes) / from 48 x 26 x
// 9 (13200): 11.9 / 11.5 / 14.3 ms.
constexpr int MG_TAIL_NODES = 4096;
// ... and most bytes of LDS for those levels' values and tables: what a CU's
// 160 KB leave beside the static arrays (33 KB with four nodes per thread).
// A level's table grows with the sum of its axes, not with its nodes, so on
// thin grids this ends the tail sooner: 4096 x 1 x 1 starts it at 1024 nodes.
constexpr int MG_TAIL_LDS = 127 * 1024;
constexpr int FIN_THREADS = 256;  // threads per instance of the solve finalizers

template <int R, bool NT, bool YZ>
__global__ void k_sweep2(const Inst *insts, const int *prefix, int ninst, int l, unsigned long long *pub,
                         unsigned seq);
template <bool YZ>
__global__ void k_seam_ring(const Inst *insts, const int *prefix, int ninst, int l);
template <int R, bool NT, bool YZ, int TY>
__global__ void k_sweep2i(const Inst *insts, const int *prefix, int ninst, int l, unsigned long long *pub,
                          unsigned seq);
template <int R, bool NT>
__global__ void k_jacobi_persist(const Inst *insts, const int *prefix, int ninst, int l0, int lcap, int ntiles);
template <int MODE, int R, bool NT, bool YZ>
__global__ void k_stencil(const Inst *insts, const int *prefix, int ninst, int l, unsigned long long *pub,
                          unsigned seq);

// Threads of k_blk: one per (x, y) column of the block with an S-node halo.
__host__ __device__ constexpr int blk_threads(int bx, int by, int s) {
    return ((bx + 2 * s) * (by + 2 * s) + 63) / 64 * 64;
}
template <int BX, int BY, int BZ, int S, int HZ, int MODE, bool YZ>
__global__ void k_blk(const Inst *insts, const int *prefix, int ninst, int l, int ns, int np, int pass,
                      unsigned long long *pub, unsigned seq);
// block shapes: X(BX, BY, BZ, S, z halo)
#define TDGL_BLK_VARIANTS(X) \
    X(16, 8, 2, 2, 2)        \
    X(32, 8, 4, 2, 2)        \
    X(32, 16, 1, 4, 0)

__global__ void k_links(const Inst *insts, int which);
__global__ void k_solve_finalize(const Inst *insts, int ninst, int count_step, int nl, int fused,
                                 unsigned long long *pub, unsigned seq);
__global__ void k_acc_reset(const Inst *insts, int ninst);
__global__ void k_jav_partial(const Inst *insts, const int *prefix, int ninst);
__global__ void k_kupdate(const Inst *insts, const int *nparts);
__global__ void k_reduce_to_state(const Inst *insts, const int *nparts, int field, int which);
__global__ void k_psi2_partial(const Inst *insts, const int *prefix, int ninst);
__global__ void k_fill_c(float2 *p, long n, float re, float im);
__global__ void k_fill_f(float *p, long n, float v);
__global__ void k_fill_u(unsigned *p, long n, unsigned v);
__global__ void k_scalars_set(const Inst *insts, int inst, StateScalars v);
__global__ void k_psi_io(const Inst *insts, int inst, float2 *ext, int to_ext);
__global__ void k_mu_io(const Inst *insts, int inst, float *ext, int to_ext);
__global__ void k_state_set(const Inst *insts, int inst, int field, double v);

__global__ void k_mg_residual(const Inst *insts, const int *prefix, int ninst, int cyc);
__global__ void k_mg_restrict(const Inst *insts, const int *prefix, int ninst, int lv, int cyc,
                              float omega);
__global__ void k_mg_prolong(const Inst *insts, const int *prefix, int ninst, int cyc);
// Blocks of k_mg_blk, and its threads: one per column of the block with its
// halo.  Runs of 192 x 101 x 33: 9.5 ms; 10.5 with 8 planes, 10.4 with 2, 10.4
// with 16 rows (the coarse levels then have too few blocks).
constexpr int MGB_X = 32, MGB_Y = 8, MGB_Z = 4;
__host__ __device__ constexpr int mgb_threads(int h) {
    return ((MGB_X + 2 * h) * (MGB_Y + 2 * h) + 63) / 64 * 64;
}
template <bool PRO, int S, bool RES>
__global__ void k_mg_blk(const Inst *insts, const int *prefix, int ninst, int lv, int isrc, int cyc, float omega);
template <int NPT, bool TL>
__global__ void k_mg_tail(const Inst *insts, int ninst, int cyc, float omega);
__global__ void k_mg_finalize(const Inst *insts, int ninst, int count_step);
__global__ void k_mu_mean_partial(const Inst *insts, const int *prefix, int ninst, int which);

// rows of the forward x transform: a real array, or the right side made from psi
enum { SRC_F = 0, SRC_PSI = 1, SRC_PSI_YZ = 2 };
template <bool P2, int XC, int SRC, bool TR>
__global__ void k_fft_fwd(const Inst *insts, const int *prefix, int ninst, const float *in_ext);
template <bool P2, int XC, bool TR>
__global__ void k_fft_inv(const Inst *insts, const int *prefix, int ninst);
template <bool P2>
__global__ void k_fft_yz(const Inst *insts, const int *prefix, int ninst);
template <bool P2>
__global__ void k_fft_y(const Inst *insts, const int *prefix, int ninst, int dir);
template <int RMAX>
__global__ void k_fft_zsolve(const Inst *insts, const int *prefix, int ninst);
__global__ void k_fft_tables(const Inst *insts, int inst);
__host__ __device__ int fft_x_pairs(int nx, int ny);
__host__ __device__ int fft_x_rows(int ny, int nz);
__host__ __device__ int fft_x_planes(int ny, int nz);
__host__ __device__ int fft_x_lds(int nx, int ny);
__host__ __device__ int fft_yz_planes(int nx, int ny, int nz);
__host__ __device__ int fft_yz_lds(int ny, int nz, int g);
__host__ __device__ int fft_y_stride(int ny);
struct FftYPlan {
    int G;       // whole planes per tile (ntk = 1)
    int ntk;     // tiles per plane (G = 1)
    int TK;      // columns per tile: G P, or about P / ntk
    int blocks;  // tiles of the instance
};
__host__ __device__ FftYPlan fft_y_plan(int nx, int ny, int nz);
__host__ __device__ int fft_pitch(int nx);
__host__ __device__ size_t fft_z_lds(int nz);
constexpr int FFT_ZTK = 16;     // kx columns per work-group of the z solve
constexpr int FFT_ZMAX = 256;   // largest nz of the spectral path
constexpr int FFT_ZSERIAL = 16; // up to this nz one lane solves a whole z system (no wavefront scan)
constexpr int FFT_MAXN = 8192;  // points per work-group of the x and y passes
constexpr int FFT_XY_THREADS = 1024;  // threads per work-group of the y passes
constexpr int FFT_X_THREADS = 256;    // threads per work-group of the x passes
constexpr int FFT_YZ_THREADS = 1024;  // threads per work-group of the fused y and z pass
constexpr int FFT_YZ_TARGET = 1024;   // its points per work-group, where several kx planes fit
constexpr int FFT_YZ_PTS = 16384;     // and at most
constexpr int FFT_YZ_BATCH = 8192;    // points it transforms at a time
constexpr int FFT_YZ_LDS = 18432;     // its LDS, complex elements (144 KB)
constexpr int FFT_X_PTS = 1024;       // complex points per work-group of the x passes (target)

constexpr int ADJ_GROUPS = 1024;  // most work-groups of the adjoint's flat passes (a multiple of 256)
__global__ void k_adj_save(const Inst *insts, float2 *dpsi, float *dmu, double *dK, int raw, double *elog);
__global__ void k_adj_load(const Inst *insts, const float2 *spsi, const float *smu, const double *sK);
__global__ void k_adj_logE(const Inst *insts, double *Elog, int n);
__global__ void k_adj_vbar(const double *Elog, int wb, int nsteps, double *vbar);
__global__ void k_adj_zero(AdjState *adj);
__global__ void k_adj_prep_f(const Inst *insts, const float *f);
__global__ void k_adj_links(const Inst *insts, const double *Kn, const double *Km, float2 *uxn);
template <bool YZ>
__global__ void k_adj_f(const Inst *insts, float2 *psibar, const float2 *psin, const float2 *uxn, double *part);
__global__ void k_adj_jterm(const Inst *insts, float2 *psibar, const float2 *psin, double *part, int have2, int kp,
                            double ew, AdjState *adj);
__global__ void k_adj_assemble(const Inst *insts, const float2 *psibar, const float2 *psim, const float *mum,
                               const float2 *lamW, const float2 *lamW_old, int extrap, const double *part,
                               AdjState *adj);
template <bool YZ>
__global__ void k_adj_sources(const Inst *insts, float2 *psibar, float *f, float *epsbar, const float2 *psim,
                              const float2 *psin, const float *mum, float2 *lamW, double *part, const AdjState *adj);

__global__ void k_incl_first(const Inst *insts, int inst, const double *centres, const double *diam,
                             int nc, unsigned *first);
__global__ void k_voronoi(const Inst *insts, int inst, const double *seeds, const float *values, int ns,
                          int metric, int axes);
__global__ void k_insulate(const Inst *insts, int inst, const unsigned char *mask);
__global__ void k_incl_first_q(const Inst *insts, int inst, const double *shapes, int nc, unsigned *first);
__global__ void k_incl_count(const unsigned *first, long N, int nc, unsigned *cnt);
__global__ void k_incl_scan(const Inst *insts, int inst, const unsigned *cnt, int nc, double target);
__global__ void k_incl_write(const Inst *insts, int inst, const unsigned *first, float eps_in,
                             float eps_out);

}  // namespace tdgl
