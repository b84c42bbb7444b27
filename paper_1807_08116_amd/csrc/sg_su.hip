// sg_su.hip -- the paper's SU kernel (Sec. 3) in its two states: the
// predictor of Eqs. (v-predictor), (e-predictor), (r-new) and the corrector
// of Eqs. (v-corrector), (e-corrector), always in FP64; the combination of
// the SPH and gravity parts into the total acceleration of Eq. (dv_dt-SPH);
// and FP64 conserved-quantity sums in a fixed reduction order.
#include "sg_internal.h"

namespace {

constexpr int kBlock = 256;
constexpr int kDiagBlocks = 512;
constexpr int kDiag = 10;

inline unsigned grid_for(int64_t n) {
    int64_t b = (n + kBlock - 1) / kBlock;
    return (unsigned)(b < 1 ? 1 : b);
}

// Predictor of particle i (Eqs. v-predictor, e-predictor, r-new).  The fused
// operations are written out here and below, so that every kernel built on
// these rounds alike.
__device__ inline void predict_one(int64_t i, int64_t ng, double dt, double* __restrict__ x,
                                   double* __restrict__ y, double* __restrict__ z,
                                   const double* __restrict__ vx, const double* __restrict__ vy,
                                   const double* __restrict__ vz, const double* __restrict__ e,
                                   const double* ax, const double* ay, const double* az,
                                   const double* __restrict__ dedt, double* __restrict__ vtx,
                                   double* __restrict__ vty, double* __restrict__ vtz,
                                   double* __restrict__ et) {
    const double hdt = 0.5 * dt;
    const double ux = vx[i], uy = vy[i], uz = vz[i];
    const double wx = __builtin_fma(dt, ax[i], ux), wy = __builtin_fma(dt, ay[i], uy),
                 wz = __builtin_fma(dt, az[i], uz);
    vtx[i] = wx;
    vty[i] = wy;
    vtz[i] = wz;
    x[i] = __builtin_fma(hdt, wx + ux, x[i]);
    y[i] = __builtin_fma(hdt, wy + uy, y[i]);
    z[i] = __builtin_fma(hdt, wz + uz, z[i]);
    if (i < ng) et[i] = __builtin_fma(dt, dedt[i], e[i]);
}

// Corrector of particle i (Eqs. v-corrector, e-corrector).
__device__ inline void correct_one(int64_t i, int64_t ng, double dt, double* __restrict__ vx,
                                   double* __restrict__ vy, double* __restrict__ vz,
                                   double* __restrict__ e, const double* __restrict__ vtx,
                                   const double* __restrict__ vty,
                                   const double* __restrict__ vtz,
                                   const double* __restrict__ et, const double* ax,
                                   const double* ay, const double* az,
                                   const double* __restrict__ dedt) {
    const double hdt = 0.5 * dt;
    vx[i] = __builtin_fma(hdt, ax[i], 0.5 * (vx[i] + vtx[i]));
    vy[i] = __builtin_fma(hdt, ay[i], 0.5 * (vy[i] + vty[i]));
    vz[i] = __builtin_fma(hdt, az[i], 0.5 * (vz[i] + vtz[i]));
    if (i < ng) e[i] = __builtin_fma(hdt, dedt[i], 0.5 * (e[i] + et[i]));
}

// a = a_SPH + g for gas (when an SPH part exists), a = g for halo.
__device__ inline void combine_one(int64_t i, int64_t ng, const double* __restrict__ asx,
                                   const double* __restrict__ asy,
                                   const double* __restrict__ asz,
                                   const double* __restrict__ gx, const double* __restrict__ gy,
                                   const double* __restrict__ gz, double* ax, double* ay,
                                   double* az) {
    double a0 = gx ? gx[i] : 0.0, a1 = gy ? gy[i] : 0.0, a2 = gz ? gz[i] : 0.0;
    if (asx && i < ng) {
        a0 += asx[i];
        a1 += asy[i];
        a2 += asz[i];
    }
    ax[i] = a0;
    ay[i] = a1;
    az[i] = a2;
}

// With PARTS, the total acceleration is formed from its parts first (and
// written to ax, ay, az): one launch and three reads a particle less than the
// combination on its own.
template <bool PARTS>
__global__ __launch_bounds__(kBlock) void k_predict(
    int64_t n, int64_t ng, double dt, double* __restrict__ x, double* __restrict__ y,
    double* __restrict__ z, const double* __restrict__ vx, const double* __restrict__ vy,
    const double* __restrict__ vz, const double* __restrict__ e, double* ax,
    double* ay, double* az, const double* __restrict__ dedt,
    double* __restrict__ vtx, double* __restrict__ vty, double* __restrict__ vtz,
    double* __restrict__ et, sg_acc_parts p) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    if (PARTS) combine_one(i, ng, p.asx, p.asy, p.asz, p.gx, p.gy, p.gz, ax, ay, az);
    predict_one(i, ng, dt, x, y, z, vx, vy, vz, e, ax, ay, az, dedt, vtx, vty, vtz, et);
}

template <bool PARTS>
__global__ __launch_bounds__(kBlock) void k_correct(
    int64_t n, int64_t ng, double dt, double* __restrict__ vx, double* __restrict__ vy,
    double* __restrict__ vz, double* __restrict__ e, const double* __restrict__ vtx,
    const double* __restrict__ vty, const double* __restrict__ vtz,
    const double* __restrict__ et, double* ax, double* ay, double* az,
    const double* __restrict__ dedt, sg_acc_parts p) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    if (PARTS) combine_one(i, ng, p.asx, p.asy, p.asz, p.gx, p.gy, p.gz, ax, ay, az);
    correct_one(i, ng, dt, vx, vy, vz, e, vtx, vty, vtz, et, ax, ay, az, dedt);
}

__global__ __launch_bounds__(kBlock) void k_combine(int64_t n, int64_t ng, sg_acc_parts p,
                                                    double* __restrict__ ax,
                                                    double* __restrict__ ay,
                                                    double* __restrict__ az) {
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    combine_one(i, ng, p.asx, p.asy, p.asz, p.gx, p.gy, p.gz, ax, ay, az);
}

// The same updates for every system of an ensemble in one launch (blocks of
// 256 particles per system), both parts of the acceleration present (SPH for
// systems with gas).
__device__ inline void seg_combine_one(const sg_seg_sys& S, int64_t i) {
    const bool sph = S.ng > 0;
    combine_one(i, S.ng, sph ? S.asx : nullptr, sph ? S.asy : nullptr, sph ? S.asz : nullptr,
                S.gx, S.gy, S.gz, S.ax, S.ay, S.az);
}

__global__ __launch_bounds__(kBlock) void k_seg_predict(const sg_seg_sys* __restrict__ sys,
                                                        const int64_t* __restrict__ pfx,
                                                        int nsys, double dt) {
    int64_t lb;
    const sg_seg_sys& S = sys[sg_seg_find(pfx, nsys, blockIdx.x, &lb)];
    const int64_t i = lb * kBlock + threadIdx.x;
    if (i >= S.n) return;
    seg_combine_one(S, i);
    predict_one(i, S.ng, dt, S.x, S.y, S.z, S.vx, S.vy, S.vz, S.e, S.ax, S.ay, S.az, S.dedt,
                S.vtx, S.vty, S.vtz, S.et);
}

__global__ __launch_bounds__(kBlock) void k_seg_correct(const sg_seg_sys* __restrict__ sys,
                                                        const int64_t* __restrict__ pfx,
                                                        int nsys, double dt) {
    int64_t lb;
    const sg_seg_sys& S = sys[sg_seg_find(pfx, nsys, blockIdx.x, &lb)];
    const int64_t i = lb * kBlock + threadIdx.x;
    if (i >= S.n) return;
    seg_combine_one(S, i);
    correct_one(i, S.ng, dt, S.vx, S.vy, S.vz, S.e, S.vtx, S.vty, S.vtz, S.et, S.ax, S.ay, S.az,
                S.dedt);
}

// Sums over the workgroup in a fixed order: each wavefront by a butterfly,
// then the four wavefronts (thread 0 holds the result).  One barrier; a tree
// through LDS component by component took 90 (final pass 12.5 -> 6 us).
__device__ inline void block_sum10(double (&v)[kDiag], double (&sh)[kBlock / 64][kDiag]) {
    for (int c = 0; c < kDiag; ++c)
        for (int o = 32; o > 0; o >>= 1) v[c] += __shfl_xor(v[c], o, 64);
    if ((threadIdx.x & 63) == 0)
        for (int c = 0; c < kDiag; ++c) sh[threadIdx.x >> 6][c] = v[c];
    __syncthreads();
    if (threadIdx.x == 0)
        for (int c = 0; c < kDiag; ++c) v[c] = (sh[0][c] + sh[1][c]) + (sh[2][c] + sh[3][c]);
}

__global__ __launch_bounds__(kBlock) void k_diag_partial(
    int64_t n, int64_t ng, const double* __restrict__ x, const double* __restrict__ y,
    const double* __restrict__ z, const double* __restrict__ vx, const double* __restrict__ vy,
    const double* __restrict__ vz, const double* __restrict__ m, const double* __restrict__ e,
    const double* __restrict__ pot, double* __restrict__ part) {
    __shared__ double sh[kBlock / 64][kDiag];
    double v[kDiag] = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    for (int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kBlock) {
        const double mi = m[i], ux = vx[i], uy = vy[i], uz = vz[i];
        const double px = x[i], py = y[i], pz = z[i];
        v[0] += 0.5 * mi * (ux * ux + uy * uy + uz * uz);
        if (i < ng) v[1] += mi * e[i];
        if (pot) v[2] += 0.5 * mi * pot[i];
        v[4] += mi * ux;
        v[5] += mi * uy;
        v[6] += mi * uz;
        v[7] += mi * (py * uz - pz * uy);
        v[8] += mi * (pz * ux - px * uz);
        v[9] += mi * (px * uy - py * ux);
    }
    block_sum10(v, sh);
    if (threadIdx.x == 0)
        for (int c = 0; c < kDiag; ++c) part[(int64_t)c * kDiagBlocks + blockIdx.x] = v[c];
}

__global__ __launch_bounds__(kBlock) void k_diag_final(const double* __restrict__ part, int nblk,
                                                       double* __restrict__ out) {
    __shared__ double sh[kBlock / 64][kDiag];
    double v[kDiag];
    for (int c = 0; c < kDiag; ++c) {
        double s = 0;
        for (int b = threadIdx.x; b < nblk; b += kBlock) s += part[c * kDiagBlocks + b];
        v[c] = s;
    }
    block_sum10(v, sh);
    if (threadIdx.x == 0) {
        for (int c = 0; c < kDiag; ++c) out[c] = v[c];
        out[3] = v[0] + v[1] + v[2];
    }
}

}  // namespace

void sg_launch_predict(int64_t n, int64_t ng, double dt, double* x, double* y, double* z,
                       const double* vx, const double* vy, const double* vz, const double* e,
                       double* ax, double* ay, double* az, const double* dedt, double* vtx,
                       double* vty, double* vtz, double* et, const sg_acc_parts* parts,
                       hipStream_t st) {
    if (parts)
        hipLaunchKernelGGL((k_predict<true>), dim3(grid_for(n)), dim3(kBlock), 0, st, n, ng, dt, x,
                           y, z, vx, vy, vz, e, ax, ay, az, dedt, vtx, vty, vtz, et, *parts);
    else
        hipLaunchKernelGGL((k_predict<false>), dim3(grid_for(n)), dim3(kBlock), 0, st, n, ng, dt,
                           x, y, z, vx, vy, vz, e, ax, ay, az, dedt, vtx, vty, vtz, et,
                           sg_acc_parts{});
}

void sg_launch_correct(int64_t n, int64_t ng, double dt, double* vx, double* vy, double* vz,
                       double* e, const double* vtx, const double* vty, const double* vtz,
                       const double* et, double* ax, double* ay, double* az, const double* dedt,
                       const sg_acc_parts* parts, hipStream_t st) {
    if (parts)
        hipLaunchKernelGGL((k_correct<true>), dim3(grid_for(n)), dim3(kBlock), 0, st, n, ng, dt,
                           vx, vy, vz, e, vtx, vty, vtz, et, ax, ay, az, dedt, *parts);
    else
        hipLaunchKernelGGL((k_correct<false>), dim3(grid_for(n)), dim3(kBlock), 0, st, n, ng, dt,
                           vx, vy, vz, e, vtx, vty, vtz, et, ax, ay, az, dedt, sg_acc_parts{});
}

void sg_launch_combine(int64_t n, int64_t ng, const sg_acc_parts& parts, double* ax, double* ay,
                       double* az, hipStream_t st) {
    hipLaunchKernelGGL(k_combine, dim3(grid_for(n)), dim3(kBlock), 0, st, n, ng, parts, ax, ay, az);
}

void sg_seg_launch_predict(const sg_seg& s, double dt, hipStream_t st) {
    if (s.nblk[SG_SEG_N] > 0)
        hipLaunchKernelGGL(k_seg_predict, dim3((unsigned)s.nblk[SG_SEG_N]), dim3(kBlock), 0, st,
                           s.sys, s.pfx + SG_SEG_N * (s.nsys + 1), s.nsys, dt);
}

void sg_seg_launch_correct(const sg_seg& s, double dt, hipStream_t st) {
    if (s.nblk[SG_SEG_N] > 0)
        hipLaunchKernelGGL(k_seg_correct, dim3((unsigned)s.nblk[SG_SEG_N]), dim3(kBlock), 0, st,
                           s.sys, s.pfx + SG_SEG_N * (s.nsys + 1), s.nsys, dt);
}

size_t sg_diag_tmp_bytes() { return sizeof(double) * kDiag * kDiagBlocks; }

void sg_launch_diagnostics(int64_t n, int64_t ng, const double* x, const double* y,
                           const double* z, const double* vx, const double* vy,
                           const double* vz, const double* m, const double* e,
                           const double* pot, double* tmp, double* out10, hipStream_t st) {
    const unsigned nb = grid_for(n) < kDiagBlocks ? grid_for(n) : kDiagBlocks;
    hipLaunchKernelGGL(k_diag_partial, dim3(nb), dim3(kBlock), 0, st, n, ng, x, y, z, vx, vy, vz,
                       m, e, pot, tmp);
    hipLaunchKernelGGL(k_diag_final, dim3(1), dim3(kBlock), 0, st, tmp, (int)nb, out10);
}
