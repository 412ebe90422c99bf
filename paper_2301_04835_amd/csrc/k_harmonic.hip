// Harmonic biasing (Sec. 2.1.1) and the samples of umbrella sampling /
// umbrella integration (Sec. 2.1.2): walker w is a window with centre
// xi0_w; its bias is sum_d k_d D_d^2 / 2 with D = xi - xi0_w (minimum image
// for a periodic CV), dV/dxi = k D, and the force -sum_d k_d D_d dxi_d/dx is
// gathered onto its atoms.  Each step may add the sample to the window's
// FP64 sums (count, sum D, sum D D^T), from which its mean and covariance
// and the mean force k (xi0 - <xi>) follow.
#include "sx_internal.h"
#include "dev_cv.h"
#include "dev_gather.h"

namespace sx {
namespace {

constexpr int kFuseBlock = 128;  // the dihedrals' wavefront and the force table's

// xi - xi0 of CV d, minimum image where it is periodic
__device__ __forceinline__ double displacement(const HarmonicArgs &a, int d, double x, double x0)
{
    double t = x - x0;
    if (a.period[d] > 0.0) t -= a.period[d] * rint(t / a.period[d]);
    return t;
}

// one workgroup per walker; thread 0 owns the window's bookkeeping and
// requests its centre and running sums before anything waits.  With FUSE
// (dihedrals, whose force table always fits the kernel arguments) thread d < D
// first evaluates dihedral d (FP64) from the positions: its value into LDS and
// the workspace, its gradient rows into LDS and the workspace's Jacobian.  The
// second wavefront requests the table's rows and the atoms' forces and forms
// the coefficients itself: after the dihedrals' barrier it only multiplies and
// stores (four dependent table loads, another barrier behind thread 0's stores
// and a trip of the gradients through L2 before: a replayed step of 256
// windows in two angles 5.8 us, now 4.7).  A kernel of two wavefronts for it
// and one of four for the others: as branches of one kernel of four, its
// registers left room for 7 of 8 wavefronts a SIMD and 2,048 windows took a
// second round (8.7 us a step; 6.6 now, 1,700 windows 6.6).
template <bool FUSE>
__global__ void __launch_bounds__(FUSE ? kFuseBlock : kBlock) k_harmonic(HarmonicArgs a)
{
    __shared__ double s_coef[kMaxCv];
    __shared__ double s_xi[kMaxBiasDim];
    __shared__ float s_J[kLdsRows][3];
    const int32_t w = blockIdx.x;
    const int u = (int)threadIdx.x - 64;
    const bool small_lane = FUSE && a.do_forces && u >= 0 && u < a.small.U;
    SmallGather sg{0.f, 0.f, 0.f, nullptr};
    int nent = 0;
    int32_t ent[kSmallPer];
    if (small_lane) small_entries(a.small, a.F, a.tabs.atom_off[w], u, sg, nent, ent);
    // thread 0's window data requested before anything waits
    double x0[kMaxBiasDim], s1p[kMaxBiasDim], s2p[kMaxBiasDim][kMaxBiasDim];
    int64_t np0 = 0;
    if (threadIdx.x == 0 || small_lane) {
#pragma unroll
        for (int d = 0; d < kMaxBiasDim; ++d) x0[d] = d < a.D ? a.xi0[(int64_t)w * a.D + d] : 0.0;
    }
    if (threadIdx.x == 0) {
#pragma unroll
        for (int d = 0; d < kMaxBiasDim; ++d) {
            s1p[d] = (a.accumulate && d < a.D) ? a.s1[(int64_t)w * a.D + d] : 0.0;
#pragma unroll
            for (int e = 0; e < kMaxBiasDim; ++e)
                s2p[d][e] = (a.accumulate && d < a.D && e < a.D) ? a.s2[((int64_t)w * a.D + d) * a.D + e] : 0.0;
        }
        if (a.accumulate) np0 = a.n[w];
    }
    if (FUSE) {
        if ((int)threadIdx.x < a.D) {
            // atom indices and slot selected by value from the kernel
            // arguments: no load between them and the positions
            int32_t at[4], slot0 = a.cs.cv[0].slot0;
#pragma unroll
            for (int q = 0; q < 4; ++q) at[q] = a.cs.cv[0].atom[q];
#pragma unroll
            for (int d = 1; d < kMaxBiasDim; ++d) {
                const bool me = (int)threadIdx.x == d;
                slot0 = me ? a.cs.cv[d].slot0 : slot0;
#pragma unroll
                for (int q = 0; q < 4; ++q) at[q] = me ? a.cs.cv[d].atom[q] : at[q];
            }
            const int64_t aoff = a.tabs.atom_off[w];
            double3 r[4], gr[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) r[q] = ld_pos(a.pos, aoff + at[q]);
            const double x = dihedral_fp64<true>(r, gr);
            s_xi[threadIdx.x] = x;
            a.xi_ws[(int64_t)w * a.D + threadIdx.x] = x;
            float *js = a.J_ws + ((int64_t)w * a.nslots + slot0) * 3;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                js[3 * q] = (float)gr[q].x;
                js[3 * q + 1] = (float)gr[q].y;
                js[3 * q + 2] = (float)gr[q].z;
                s_J[slot0 + q][0] = (float)gr[q].x;
                s_J[slot0 + q][1] = (float)gr[q].y;
                s_J[slot0 + q][2] = (float)gr[q].z;
            }
        }
        __syncthreads();  // s_xi and s_J
    }
    if (small_lane) {
        double coef[kMaxBiasDim] = {0.0, 0.0, 0.0};
#pragma unroll
        for (int d = 0; d < kMaxBiasDim; ++d)
            if (d < a.D) coef[d] = -(a.k[d] * displacement(a, d, s_xi[d], x0[d]));
        float jr[kSmallPer][3];
        small_jacobian(&s_J[0][0], ent, jr);
        small_forces(a.small, a.F, sg, nent, ent, jr, coef);
    }
    if (threadIdx.x == 0) {
        double Dv[kMaxBiasDim], V = 0.0;
        bool finite = true;
#pragma unroll
        for (int d = 0; d < kMaxBiasDim; ++d) {
            if (d >= a.D) break;
            const double x = FUSE ? s_xi[d] : a.xi[(int64_t)w * a.D + d];
            const double t = displacement(a, d, x, x0[d]);
            Dv[d] = t;
            const double g = a.k[d] * t;
            V += 0.5 * g * t;
            finite = finite && isfinite(g);
            a.dV_ws[(int64_t)w * a.D + d] = g;
            if (a.dV_out) a.dV_out[(int64_t)w * a.D + d] = g;
            if (a.xi_out) a.xi_out[(int64_t)w * a.D + d] = x;
            s_coef[d] = -g;
        }
        a.V_ws[w] = V;
        if (a.V_out) a.V_out[w] = V;
        if (!finite || !isfinite(V)) atomicOr(a.flags, kFlagNonFinite);
        if (a.accumulate) {
            a.n[w] = np0 + 1;
#pragma unroll
            for (int d = 0; d < kMaxBiasDim; ++d) {
                if (d >= a.D) break;
                a.s1[(int64_t)w * a.D + d] = s1p[d] + Dv[d];
#pragma unroll
                for (int e = 0; e < kMaxBiasDim; ++e)
                    if (e < a.D) a.s2[((int64_t)w * a.D + d) * a.D + e] = s2p[d][e] + Dv[d] * Dv[e];
            }
        }
        if (w == 0 && a.count_step) *a.dstep = a.step >= 0 ? a.step + 1 : *a.dstep + 1;
    }
    if (FUSE) return;
    __syncthreads();
    if (a.do_forces) gather_forces(a.tabs, a.J + (int64_t)w * a.nslots * 3, w, s_coef, a.F);
}

}  // namespace

hipError_t launch_harmonic(const HarmonicArgs &a, hipStream_t s)
{
    if (a.tabs.W < 1) return hipErrorInvalidValue;
    if (a.fuse_cv && (!a.small.on || a.nslots > kLdsRows)) return hipErrorInvalidValue;
    if (a.fuse_cv)
        hipLaunchKernelGGL(k_harmonic<true>, dim3(a.tabs.W), dim3(kFuseBlock), 0, s, a);
    else
        hipLaunchKernelGGL(k_harmonic<false>, dim3(a.tabs.W), dim3(kBlock), 0, s, a);
    return hipGetLastError();
}

}  // namespace sx
