// Metadynamics bias kept on a grid (Sec. 2.1.5: the bias may be stored on a
// pre-defined grid, trading accuracy for speed).  Each hill list has a grid
// holding, at every node, the list's bias V and its gradient dV/dxi; a CV
// value reads them back by multilinear interpolation over the 2^D nodes of
// its cell (V and each gradient component interpolated on their own).
// Outside the range of a non-periodic CV there is no bias.
//
//   k_grid_step     one workgroup per walker: the read-back, the outputs, the
//                   well-tempered deposit into the hill list (height from
//                   the read-back V) and the force gather; k_grid_step_wave
//                   is the same in one wavefront when forces go through the
//                   table in kernel-argument form.
//   k_grid_tiles, k_grid_line, k_grid_fill, k_grid_few
//                   the hills the step appended, or a whole list (rebuild, in
//                   slices that k_grid_join adds up), onto every node; after
//                   a step the list's count and the device step counter
//                   advance.
//   k_grid_eval     the read-back at arbitrary points.
//
// Node sums run in FP64 in a fixed order, so a grid holds the exact hill sum
// at its nodes up to the rounding of its factors.
#include "sx_internal.h"
#include "dev_cv.h"
#include "dev_gather.h"

namespace sx {
namespace {

// The cell of xi: lower and upper node per CV and the fractions t; false
// outside the range of a non-periodic CV (its nodes are then set to 0).
__device__ __forceinline__ bool grid_cell(const GridArgs &g, const double *xi, int32_t (&i0)[kMaxBiasDim],
                                          int32_t (&i1)[kMaxBiasDim], double (&t)[kMaxBiasDim])
{
    bool inside = true;
#pragma unroll
    for (int d = 0; d < kMaxBiasDim; ++d) {  // compile-time indices, all of them set (registers)
        i0[d] = i1[d] = 0;
        t[d] = 0.0;
        if (d >= g.D) continue;
        const double u = (xi[d] - g.lo[d]) / g.delta[d];
        double fl = floor(u);
        t[d] = u - fl;
        if (g.per[d]) {
            int64_t k = (int64_t)fl % g.nbins[d];
            if (k < 0) k += g.nbins[d];
            i0[d] = (int32_t)k;
            i1[d] = i0[d] + 1 == g.nbins[d] ? 0 : i0[d] + 1;
        } else {
            if (!(u >= 0.0 && u <= (double)g.nbins[d])) {
                inside = false;
                continue;
            }
            int32_t k = (int32_t)fl;
            if (k == g.nbins[d]) {  // xi == hi: the last cell, weight 1 on its far node
                k = g.nbins[d] - 1;
                t[d] = 1.0;
            }
            i0[d] = k;
            i1[d] = k + 1;
        }
    }
    return inside;
}

// Corner c of the cell: its node index and multilinear weight.  Corner c
// takes node i1 of CV d when bit D - 1 - d of c is set (first CV the most
// significant).
__device__ __forceinline__ int64_t grid_corner(const GridArgs &g, int c, const int32_t (&i0)[kMaxBiasDim],
                                               const int32_t (&i1)[kMaxBiasDim], const double (&t)[kMaxBiasDim],
                                               double &wgt)
{
    int64_t idx = 0;
    wgt = 1.0;
#pragma unroll
    for (int d = 0; d < kMaxBiasDim; ++d) {
        if (d >= g.D) continue;
        const bool hi = (c >> (g.D - 1 - d)) & 1;
        const int32_t n0 = i0[d], n1 = i1[d];  // select values, not addresses (keeps the arrays in registers)
        idx = idx * g.n[d] + (hi ? n1 : n0);
        wgt *= hi ? t[d] : 1.0 - t[d];
    }
    return idx;
}

// The interpolated (V, dV/dxi) of grid l at xi, corners summed in order;
// false (and zeros) outside the range of a non-periodic CV.
__device__ bool grid_read(const GridArgs &g, int32_t l, const double *xi, double &V, double (&G)[kMaxBiasDim])
{
    int32_t i0[kMaxBiasDim], i1[kMaxBiasDim];
    double t[kMaxBiasDim];
    const bool inside = grid_cell(g, xi, i0, i1, t);
    V = 0.0;
    for (int d = 0; d < kMaxBiasDim; ++d) G[d] = 0.0;
    if (!inside) return false;
    const double *Vg = g.V + (int64_t)l * g.N;
    const double *Gg = g.G + (int64_t)l * g.D * g.N;
    for (int c = 0; c < (1 << g.D); ++c) {
        double wgt;
        const int64_t idx = grid_corner(g, c, i0, i1, t, wgt);
        V += wgt * Vg[idx];
#pragma unroll
        for (int d = 0; d < kMaxBiasDim; ++d)
            if (d < g.D) G[d] += wgt * Gg[(int64_t)d * g.N + idx];
    }
    return true;
}

__global__ void __launch_bounds__(kBlock) k_grid_step(GridArgs g)
{
    __shared__ double s_coef[kMaxCv];
    const int32_t w = blockIdx.x;
    const int32_t l = g.shared ? 0 : w;
    if (threadIdx.x == 0) {
        double xi[kMaxBiasDim], V, G[kMaxBiasDim];
        for (int d = 0; d < g.D; ++d) xi[d] = g.xi[(int64_t)w * g.D + d];
        const bool inside = grid_read(g, l, xi, V, G);
        bool finite = isfinite(V);
        g.V_ws[w] = V;
        if (g.V_out) g.V_out[w] = V;
        for (int d = 0; d < g.D; ++d) {
            finite = finite && isfinite(G[d]);
            g.dV_ws[(int64_t)w * g.D + d] = G[d];
            if (g.dV_out) g.dV_out[(int64_t)w * g.D + d] = G[d];
            if (g.xi_out) g.xi_out[(int64_t)w * g.D + d] = xi[d];
            s_coef[d] = -G[d];
        }
        if (!finite) atomicOr(g.flags, kFlagNonFinite);
        // the step number after this one: the step kernel reads the device
        // counter (only where a deposit depends on it), the add kernel that
        // follows advances it
        bool dep = g.deposit == 2;
        if (g.deposit == 1 && g.stride > 0) {
            const int64_t next_step = g.step >= 0 ? g.step + 1 : *g.dstep + 1;
            dep = (next_step - 1) % g.stride == 0;
        }
        if (dep && (inside || g.shared)) {
            // outside the grid nothing is deposited, except that a walker
            // keeps its slot of a shared list (walker order) with a hill of
            // height 0, which adds nothing to the bias
            const double h = !inside ? 0.0 : g.inv_kdT > 0.0 ? g.height * exp(-V * g.inv_kdT) : g.height;
            const WalkerRec wr = g.wrec[l];
            const int64_t hb = (int64_t)wr.hb4 * 4;
            const int32_t cnt = g.count[l];
            const int32_t nnew = g.shared ? g.tabs.W : 1;
            if ((int64_t)cnt + nnew <= wr.cap) {
                const int64_t k = hb + cnt + (g.shared ? w : 0);
                for (int d = 0; d < g.D; ++d) g.c[d][k] = (float)xi[d];
                g.h[k] = (float)h;
                if (!g.shared || w == 0) g.pend[l] = nnew;
            } else {
                atomicOr(g.flags, kFlagCapacity);
            }
        }
    }
    __syncthreads();
    if (g.count_in_step && w == 0 && threadIdx.x == 0) *g.dstep = g.step >= 0 ? g.step + 1 : *g.dstep + 1;
    if (g.do_forces) gather_forces(g.tabs, g.J + (int64_t)w * g.nslots * 3, w, s_coef, g.F);
}

// The same step in one wavefront, for steps that gather forces through the
// table in kernel-argument form.  Every lane finds the cell (the same
// values), lane c < 2^D loads corner c's V and dV/dxi, and every lane sums
// the corner terms in corner order through shuffles (the serial order and
// bits of grid_read); xi, the list's count and record and each lane's table
// row with its Jacobian rows and force are requested before any wait (lanes
// past 2^D or U re-read corner 0 or row U - 1 and drop it).  Lane 0 writes
// the outputs and deposits, lane u < U adds atom u's force.
__global__ void __launch_bounds__(64) k_grid_step_wave(GridArgs g)
{
    __shared__ float s_J[kLdsRows][3];  // fused CVs: the walker's Jacobian slots
    const int32_t w = blockIdx.x;
    const int32_t l = g.shared ? 0 : w;
    const int lane = threadIdx.x;
    const bool dep_cnt = g.deposit == 1 && g.stride > 0;
    const int64_t dstep = dep_cnt && g.step < 0 ? *g.dstep : 0;
    const int32_t cnt = g.deposit ? g.count[l] : 0;
    // no deposit in this configuration: the counter moves here (nothing reads it in this kernel)
    if (g.count_in_step && w == 0 && lane == 0) *g.dstep = g.step >= 0 ? g.step + 1 : *g.dstep + 1;
    const WalkerRec wr = g.wrec[l];
    const int64_t aoff = g.tabs.atom_off[w];
    SmallGather sg{0.f, 0.f, 0.f, nullptr};
    int nent = 0;
    int32_t ent[kSmallPer];
    float jr[kSmallPer][3];
    double xi[kMaxBiasDim];
    if (g.fuse_cv) {
        // this lane's table row and force (the Jacobian rows come from LDS),
        // ahead of the dihedrals
        small_entries(g.small, g.F, aoff, min(lane, g.small.U - 1), sg, nent, ent);
        // lane d < D evaluates dihedral d of the walker in FP64 (atom indices
        // and slots selected from the kernel arguments by value); its value
        // goes to every lane, its four gradient rows to LDS and the workspace
        int32_t at[4], slot0 = g.cs.cv[0].slot0;
#pragma unroll
        for (int q = 0; q < 4; ++q) at[q] = g.cs.cv[0].atom[q];
#pragma unroll
        for (int d = 1; d < kMaxBiasDim; ++d)
            if (lane == d && d < g.D) {
                slot0 = g.cs.cv[d].slot0;
#pragma unroll
                for (int q = 0; q < 4; ++q) at[q] = g.cs.cv[d].atom[q];
            }
        double xd = 0.0;
        if (lane < g.D) {
            double3 r[4], gr[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) r[q] = ld_pos(g.pos, aoff + at[q]);
            xd = dihedral_fp64<true>(r, gr);
            g.xi_ws[(int64_t)w * g.D + lane] = xd;
            float *js = g.J_ws + ((int64_t)w * g.nslots + slot0) * 3;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float gx = (float)gr[q].x, gy = (float)gr[q].y, gz = (float)gr[q].z;
                js[3 * q] = gx;
                js[3 * q + 1] = gy;
                js[3 * q + 2] = gz;
                s_J[slot0 + q][0] = gx;
                s_J[slot0 + q][1] = gy;
                s_J[slot0 + q][2] = gz;
            }
        }
#pragma unroll
        for (int d = 0; d < kMaxBiasDim; ++d) xi[d] = __shfl(xd, min(d, g.D - 1), 64);
        __syncthreads();  // s_J written (one wavefront)
        small_jacobian(&s_J[0][0], ent, jr);  // slot < 4 D: every CV a dihedral
    } else {
        // xi over the largest CV count with the index clamped to the last
        // CV (in bounds, the extra entries unused), so the loads are issued
        // together
#pragma unroll
        for (int d = 0; d < kMaxBiasDim; ++d) xi[d] = g.xi[(int64_t)w * g.D + min(d, g.D - 1)];
        small_rows(g.small, g.J + (int64_t)w * g.nslots * 3, g.F, aoff, min(lane, g.small.U - 1), sg, nent, ent, jr);
    }
    int32_t i0[kMaxBiasDim], i1[kMaxBiasDim];
    double t[kMaxBiasDim];
    const bool inside = grid_cell(g, xi, i0, i1, t);
    const int nc = 1 << g.D;
    double wgt;
    const int64_t idx = grid_corner(g, lane < nc ? lane : 0, i0, i1, t, wgt);
    const double *Vg = g.V + (int64_t)l * g.N;
    const double *Gg = g.G + (int64_t)l * g.D * g.N;
    const double tv = wgt * Vg[idx];
    double tg[kMaxBiasDim];
#pragma unroll
    for (int d = 0; d < kMaxBiasDim; ++d) tg[d] = d < g.D ? wgt * Gg[(int64_t)min(d, g.D - 1) * g.N + idx] : 0.0;
    double V = 0.0, G[kMaxBiasDim] = {0.0, 0.0, 0.0};
    for (int c = 0; c < nc; ++c) {
        V += __shfl(tv, c, 64);
        for (int d = 0; d < kMaxBiasDim; ++d) G[d] += __shfl(tg[d], c, 64);
    }
    if (!inside) {
        V = 0.0;
        for (int d = 0; d < kMaxBiasDim; ++d) G[d] = 0.0;
    }
    // ahead of lane 0's outputs, whose arithmetic then overlaps these stores
    if (lane < g.small.U) {
        double coef[kMaxBiasDim];
#pragma unroll
        for (int d = 0; d < kMaxBiasDim; ++d) coef[d] = -G[d];
        small_forces(g.small, g.F, sg, nent, ent, jr, coef);
    }
    if (lane == 0) {
        bool finite = isfinite(V);
        g.V_ws[w] = V;
        if (g.V_out) g.V_out[w] = V;
#pragma unroll
        for (int d = 0; d < kMaxBiasDim; ++d) {
            if (d >= g.D) continue;
            finite = finite && isfinite(G[d]);
            g.dV_ws[(int64_t)w * g.D + d] = G[d];
            if (g.dV_out) g.dV_out[(int64_t)w * g.D + d] = G[d];
            if (g.xi_out) g.xi_out[(int64_t)w * g.D + d] = xi[d];
        }
        if (!finite) atomicOr(g.flags, kFlagNonFinite);
        const int64_t next_step = g.step >= 0 ? g.step + 1 : dstep + 1;
        bool dep = g.deposit == 2;
        if (dep_cnt) dep = (next_step - 1) % g.stride == 0;
        if (dep && (inside || g.shared)) {  // as k_grid_step
            const double h = !inside ? 0.0 : g.inv_kdT > 0.0 ? g.height * exp(-V * g.inv_kdT) : g.height;
            const int64_t hb = (int64_t)wr.hb4 * 4;
            const int32_t nnew = g.shared ? g.tabs.W : 1;
            if ((int64_t)cnt + nnew <= wr.cap) {
                const int64_t k = hb + cnt + (g.shared ? w : 0);
#pragma unroll
                for (int d = 0; d < kMaxBiasDim; ++d)
                    if (d < g.D) g.c[d][k] = (float)xi[d];
                g.h[k] = (float)h;
                if (!g.shared || w == 0) g.pend[l] = nnew;
            } else {
                atomicOr(g.flags, kFlagCapacity);
            }
        }
    }
}

// ---------------------------------------------------- hills onto the nodes
// A hill's Gaussian is a product of one factor per CV, so over a block of
// nodes the sums over hills are matrix products.  With the nodes' last CV as
// columns and the CVs before it as rows, and per hill k
//   L0(r) = h_k prod_{d < D-1} e_d,  R0(c) = e_{D-1},  e_d = exp(-u_d^2/2s_d^2),
//   g_d = -u_d / s_d^2,  u_d = node - centre (minimum image),
//   V += sum_k L0 R0,  G_d += sum_k (L0 g_d) R0 (d < D-1),  G_{D-1} += sum_k L0 (R0 g_{D-1}).
//
// k_grid_tiles (D >= 2): a workgroup owns a tile of 32 x 32 nodes; KG groups
// of four wavefronts take 16 hills at a time, form the tile's 32 row and 32
// column factors in LDS (64 exponentials for 1024 nodes) and multiply them
// with v_mfma_f64_16x16x4_f64, each wavefront a 16 x 16 block of the 1 + D
// sums; the groups' sums are joined in group order and added to the nodes, so
// a grid's bits do not depend on the schedule.  FP64 multiply-adds bound it
// (1 + D per (node, hill), 39 T/s), and the factors' exponentials (about 40
// operations each, 1/16 per (node, hill)), which do not run beside them.
// A whole list takes KG = 4 (16 wavefronts a CU) and as many slices as fill the
// chip, a step's few hills KG = 1: less to launch on the many steps that
// deposit nothing.  256 hills: 25 us (one workgroup for the whole grid:
// 76.8 ms).  KG = 4 spills 42 registers in two CVs and 70 in three; KG = 2 none,
// but is no faster (30,000 hills onto 24 x 24 x 24 nodes 279 us, 250 with four;
// 100 x 100 x 3 2,753 and 2,464; 30 x 30 x 20 339 and 376).
//
// k_grid_fill: a whole list in tiles of 64 x 64, half the factors per node.
// 100,000 hills onto 512 x 512 nodes, upload included: 3.42 ms; in 32 x 32
// tiles 4.4, with one exponential and two divisions per (node, hill) and one
// lane per node 121.  The matrix units' FP64 rate and the factors, which do
// not overlap, bound it: 2.1 and 0.9 ms.
//
// k_grid_line (D = 1): no product to share, one exponential per (node, hill);
// a wavefront per 64 nodes and sixteenth of the hills, four of them requested
// at a time, the sixteen sums joined in order.
typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr int kTileSide = 32;   // nodes of a tile per side
constexpr int kTileHills = 16;  // hills per stage of a group
// LDS row stride (doubles): the four hills of a fragment start 32 banks apart
constexpr int kTileLd = 48;
constexpr int kLineSlices = 16;
constexpr int kFillSide = 64;   // nodes per side of a rebuild's larger tile
// The larger tile's time in tenths of a 32 x 32 tile's.  60,000 hills, ms: 512 x
// 512 nodes 2.06 in 64 tiles, 2.67 in 256 (31); 48 x 48 x 48 1.63 in 36, 2.16 in
// 144 (30); 200 x 200 in 16 and 49 even (0.64 and 0.62; 30,000 hills 0.325 and
// 0.342).
constexpr int kFillCost = 30;
constexpr int kMostSlices = 128;

// 2^y for y <= 0 in FP64: y = n + f, |f| <= 1/2, and the Taylor series of
// exp(f ln 2) to degree 13 (remainder below 5e-18), scaled by 2^n.  About
// half the operations of exp(), whose other half serves arguments that do
// not occur here; below 2^-1100 (and for y = -inf) the scaling gives 0, NaN
// stays NaN.
__device__ __forceinline__ double exp2_neg(double y)
{
    const double yc = y < -1100.0 ? -1100.0 : y;
    const double n = rint(yc), f = yc - n;
    double p = 1.3691488853904128880892e-12;  // ln2^13 / 13!, then down to ln2^0 / 0!
    p = fma(p, f, 2.5678435993488205141995e-11);
    p = fma(p, f, 4.4455382718708114975964e-10);
    p = fma(p, f, 7.0549116208011233298754e-9);
    p = fma(p, f, 1.0178086009239699727491e-7);
    p = fma(p, f, 1.3215486790144309488404e-6);
    p = fma(p, f, 1.5252733804059840280026e-5);
    p = fma(p, f, 1.5403530393381609954437e-4);
    p = fma(p, f, 1.3333558146428443423412e-3);
    p = fma(p, f, 9.6181291076284771619791e-3);
    p = fma(p, f, 5.5504108664821579953142e-2);
    p = fma(p, f, 2.4022650695910071233355e-1);
    p = fma(p, f, 6.9314718055994530941723e-1);
    p = fma(p, f, 1.0);
    return ldexp(p, (int)n);
}

// The displacement u = x - c of CV d.  Its image is that of rint(u / period):
// where the product with the reciprocal is too near half a period to tell, the
// quotient decides.  In the units of exp2_neg: y = -u^2 / (2 sigma^2 ln 2).
__device__ __forceinline__ double axis_offset(const GridArgs &g, int d, double x, double c, double &y)
{
    double u = x - c;
    if (g.period[d] > 0.0) {
        double v = fma(-g.period[d], rint(u * g.inv_period[d]), u);
        if (__builtin_expect(fabs(v) > 0.499999999 * g.period[d], 0)) v = fma(-g.period[d], rint(u / g.period[d]), u);
        u = v;
    }
    y = -(u * u) * (0.72134752044448170368 * g.inv_sig2[d]);  // log2(e) / 2
    return u;
}

// the factor e of CV d at displacement u, and g = -u / sigma^2
__device__ __forceinline__ void axis_factor(const GridArgs &g, int d, double x, double c, double &e, double &gd)
{
    double y;
    gd = -axis_offset(g, d, x, c, y) * g.inv_sig2[d];
    e = exp2_neg(y);
}

// The hills [k0, k1) of grid l that a workgroup sums: after k_grid_step the
// `pend` hills behind the count (none on most steps), in a rebuild its slice
// of the whole list.
template <bool REBUILD>
__device__ __forceinline__ void hill_range(const GridArgs &g, int32_t l, int32_t slice, int32_t &k0, int32_t &k1)
{
    const int32_t cnt = g.count[l];
    if (REBUILD) {
        const int32_t per = (cnt + g.slices - 1) / g.slices;
        k0 = (int32_t)min((int64_t)cnt, (int64_t)slice * per);
        k1 = min(cnt, k0 + per);
    } else {
        k0 = cnt;
        k1 = cnt + g.pend[l];
    }
}

// Where a workgroup's sums go: grid l, or its slice's record of a rebuild.
template <bool REBUILD>
__device__ __forceinline__ void node_sums(const GridArgs &g, int32_t l, int32_t slice, double *&Vg, double *&Gg)
{
    const bool record = REBUILD && g.slices > 1;
    Vg = record ? g.part + (int64_t)slice * (1 + g.D) * g.N : g.V + (int64_t)l * g.N;
    Gg = record ? Vg + g.N : g.G + (int64_t)l * g.D * g.N;
}

// The end of a step's launch on grid l: the last of the list's workgroups to
// arrive moves the count past the new hills.  Every workgroup has then read
// count and pend (its ticket follows its use of them), and nothing it wrote
// is read before the next launch, so the ticket orders no other memory.
__device__ __forceinline__ void finish_add(const GridArgs &g, int32_t l, int32_t k1, int32_t per)
{
    if (threadIdx.x != 0) return;
    if (atomicAdd(&g.tick[l], 1) != per - 1) return;
    g.count[l] = k1;
    g.pend[l] = 0;
    g.tick[l] = 0;
}

// the step counter moves here (nothing else of the launch reads it)
__device__ __forceinline__ void advance_step(const GridArgs &g)
{
    if (g.count_step && blockIdx.x == 0 && threadIdx.x == 0)
        *g.dstep = g.step >= 0 ? g.step + 1 : *g.dstep + 1;
}

template <int D, int KG, bool REBUILD>
__global__ void __launch_bounds__(256 * KG) k_grid_tiles(GridArgs g, int32_t l0, int32_t per)
{
    __shared__ double s_f[KG][D + 2][kTileHills][kTileLd];  // L0, L0 g_0 .., then R0, R0 g_last
    if (!REBUILD) advance_step(g);
    const int32_t z = (int32_t)blockIdx.x / per, wg = (int32_t)blockIdx.x % per;  // per workgroups a grid or slice
    const int32_t l = REBUILD ? l0 : z, slice = REBUILD ? z : 0;
    int32_t k0, k1;
    hill_range<REBUILD>(g, l, slice, k0, k1);
    if (!REBUILD && k1 == k0) return;  // uniform
    const int grp = threadIdx.x >> 8, t = threadIdx.x & 255;
    const int lane = t & 63, wr = (t >> 7) & 1, wc = (t >> 6) & 1;  // this wavefront's 16 x 16 block
    const int64_t nc = g.n[D - 1], nr = g.N / nc;
    const int64_t tc = (nc + kTileSide - 1) / kTileSide, tiles = tc * ((nr + kTileSide - 1) / kTileSide);
    const int64_t hb = (int64_t)g.wrec[l].hb4 * 4;
    double *Vg, *Gg;
    node_sums<REBUILD>(g, l, slice, Vg, Gg);
    const int fh = t >> 4, fq = t & 15;  // factors: hill fh of the stage, rows and columns fq, fq + 16
    for (int64_t tile = wg; tile < tiles; tile += per) {
        const int64_t r0 = tile / tc * kTileSide, c0 = tile % tc * kTileSide;
        double xr[2][D - 1], xc[2];
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            int64_t r = r0 + fq + 16 * q;
#pragma unroll
            for (int d = D - 2; d >= 0; --d) {
                xr[q][d] = g.lo[d] + (double)(r % g.n[d]) * g.delta[d];
                r /= g.n[d];
            }
            const int64_t c = c0 + fq + 16 * q;
            xc[q] = g.lo[D - 1] + (double)c * g.delta[D - 1];
        }
        f64x4 acc[1 + D];  // V, G_0 .. G_{D-1}
#pragma unroll
        for (int q = 0; q <= D; ++q) acc[q] = f64x4{0.0, 0.0, 0.0, 0.0};
        // the group's next hill of this lane, requested a stage ahead
        float hc[D], hh = 0.f;
        auto request = [&](int32_t k) {
            const int64_t at = hb + (k < k1 ? k : k0);
#pragma unroll
            for (int d = 0; d < D; ++d) hc[d] = g.c[d][at];
            hh = g.h[at];
        };
        // the factors of the group's stage at hill kb.  A hill past the range
        // takes zero height on the first hill's centre; rows and columns past
        // the grid are formed and not stored.
        auto factors = [&](int32_t kb) {
            const double h = kb + fh < k1 ? (double)hh : 0.0;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                double L = h, gd[D - 1], e, gl;
#pragma unroll
                for (int d = 0; d < D - 1; ++d) {
                    axis_factor(g, d, xr[q][d], (double)hc[d], e, gd[d]);
                    L *= e;
                }
                s_f[grp][0][fh][fq + 16 * q] = L;
#pragma unroll
                for (int d = 0; d < D - 1; ++d) s_f[grp][1 + d][fh][fq + 16 * q] = L * gd[d];
                axis_factor(g, D - 1, xc[q], (double)hc[D - 1], e, gl);
                s_f[grp][D][fh][fq + 16 * q] = e;
                s_f[grp][D + 1][fh][fq + 16 * q] = e * gl;
            }
            request(kb + KG * kTileHills + fh);
        };
        auto products = [&]() {
#pragma unroll
            for (int ks = 0; ks < kTileHills / 4; ++ks) {
                const int kk = 4 * ks + (lane >> 4), a = 16 * wr + (lane & 15), b = 16 * wc + (lane & 15);
                const double l0v = s_f[grp][0][kk][a], e0 = s_f[grp][D][kk][b];
                acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(l0v, e0, acc[0], 0, 0, 0);
#pragma unroll
                for (int d = 0; d < D - 1; ++d)
                    acc[1 + d] = __builtin_amdgcn_mfma_f64_16x16x4f64(s_f[grp][1 + d][kk][a], e0, acc[1 + d], 0, 0, 0);
                acc[D] = __builtin_amdgcn_mfma_f64_16x16x4f64(l0v, s_f[grp][D + 1][kk][b], acc[D], 0, 0, 0);
            }
        };
        const int32_t stages = (k1 - k0 + KG * kTileHills - 1) / (KG * kTileHills);
        const int32_t kg0 = k0 + grp * kTileHills;
        if (stages > 0) request(kg0 + fh);
        for (int32_t i = 0; i < stages; ++i) {
            factors(kg0 + i * KG * kTileHills);
            __syncthreads();
            products();
            __syncthreads();
        }
        if (KG > 1) {  // join the groups' sums, group after group
            double *red = &s_f[0][0][0][0];  // (KG - 1) x (1 + D) x 1024 doubles
            static_assert((KG - 1) * (1 + D) * 1024 <= KG * (D + 2) * kTileHills * kTileLd, "LDS reuse");
            if (grp > 0) {
#pragma unroll
                for (int q = 0; q <= D; ++q)
#pragma unroll
                    for (int v = 0; v < 4; ++v) red[(((grp - 1) * (1 + D) + q) * 4 + v) * 256 + t] = acc[q][v];
            }
            __syncthreads();
            if (grp == 0) {
#pragma unroll
                for (int o = 0; o < KG - 1; ++o)
#pragma unroll
                    for (int q = 0; q <= D; ++q)
#pragma unroll
                        for (int v = 0; v < 4; ++v) acc[q][v] += red[((o * (1 + D) + q) * 4 + v) * 256 + t];
            }
        }
        if (grp == 0) {
            // lane: column lane % 16, rows lane / 16 + 4 v of its block
            const int64_t c = c0 + 16 * wc + (lane & 15);
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int64_t r = r0 + 16 * wr + (lane >> 4) + 4 * v;
                if (r >= nr || c >= nc) continue;
                const int64_t node = r * nc + c;
                Vg[node] = REBUILD ? acc[0][v] : Vg[node] + acc[0][v];
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    double *p = Gg + (int64_t)d * g.N + node;
                    *p = REBUILD ? acc[1 + d][v] : *p + acc[1 + d][v];
                }
            }
        }
        __syncthreads();  // s_f is free for the next tile
    }
    if (!REBUILD) finish_add(g, l, k1, per);
}

template <bool REBUILD>
__global__ void __launch_bounds__(64 * kLineSlices) k_grid_line(GridArgs g, int32_t l0, int32_t per)
{
    __shared__ double s_r[kLineSlices][2][64];
    if (!REBUILD) advance_step(g);
    const int32_t z = (int32_t)blockIdx.x / per, wg = (int32_t)blockIdx.x % per;  // per workgroups a grid or slice
    const int32_t l = REBUILD ? l0 : z, slice = REBUILD ? z : 0;
    int32_t k0, k1;
    hill_range<REBUILD>(g, l, slice, k0, k1);
    if (!REBUILD && k1 == k0) return;  // uniform
    const int lane = threadIdx.x & 63, sub = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t hb = (int64_t)g.wrec[l].hb4 * 4;
    double *Vg, *Gg;
    node_sums<REBUILD>(g, l, slice, Vg, Gg);
    for (int64_t n0 = (int64_t)wg * 64; n0 < g.N; n0 += (int64_t)per * 64) {
        const int64_t node = n0 + lane;
        const double x = g.lo[0] + (double)node * g.delta[0];
        double v = 0.0, gr = 0.0;
        // four of the wavefront's hills requested together; one past the range
        // takes zero height on the first hill's centre
        for (int32_t k = k0 + sub; k < k1; k += 4 * kLineSlices) {
            float c[4], h[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t at = hb + (k + q * kLineSlices < k1 ? k + q * kLineSlices : k0);
                c[q] = g.c[0][at];
                h[q] = g.h[at];
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                double e, gd;
                axis_factor(g, 0, x, (double)c[q], e, gd);
                e *= k + q * kLineSlices < k1 ? (double)h[q] : 0.0;
                v += e;
                gr = fma(e, gd, gr);
            }
        }
        s_r[sub][0][lane] = v;
        s_r[sub][1][lane] = gr;
        __syncthreads();
        if (sub == 0 && node < g.N) {
            for (int q = 1; q < kLineSlices; ++q) {
                v += s_r[q][0][lane];
                gr += s_r[q][1][lane];
            }
            Vg[node] = REBUILD ? v : Vg[node] + v;
            Gg[node] = REBUILD ? gr : Gg[node] + gr;
        }
        __syncthreads();  // s_r is free for the next nodes
    }
    if (!REBUILD) finish_add(g, l, k1, per);
}

// A rebuild's sums of 64 x 64 nodes (D >= 2): the 16 wavefronts of a workgroup
// take the same 16 hills, one each for the 64 row and 64 column factors (half
// as many exponentials per node as a 32 x 32 tile), then a 16 x 16 block of the
// products each.  Two stages of factors in LDS: one barrier a stage, and a
// wavefront forms its next factors without waiting for the others' products.
template <int D>
__global__ void __launch_bounds__(1024) k_grid_fill(GridArgs g, int32_t l, int32_t tiles)
{
    constexpr int Ld = kFillSide + 16;  // as kTileLd
    __shared__ double s_f[2][D + 2][kTileHills][Ld];
    const int32_t slice = (int32_t)blockIdx.x / tiles, tile = (int32_t)blockIdx.x % tiles;
    int32_t k0, k1;
    hill_range<true>(g, l, slice, k0, k1);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t nc = g.n[D - 1], nr = g.N / nc;
    const int32_t tc = (int32_t)((nc + kFillSide - 1) / kFillSide);
    const int64_t r0 = (int64_t)(tile / tc) * kFillSide, c0 = (int64_t)(tile % tc) * kFillSide;
    const int64_t hb = (int64_t)g.wrec[l].hb4 * 4;
    // rows and columns past the grid are formed and not stored
    double xr[D - 1];
    int64_t rr = r0 + lane;
#pragma unroll
    for (int d = D - 2; d >= 0; --d) {
        xr[d] = g.lo[d] + (double)(rr % g.n[d]) * g.delta[d];
        rr /= g.n[d];
    }
    const double xc = g.lo[D - 1] + (double)(c0 + lane) * g.delta[D - 1];
    f64x4 acc[1 + D];
#pragma unroll
    for (int q = 0; q <= D; ++q) acc[q] = f64x4{0.0, 0.0, 0.0, 0.0};
    // the wavefront's hill of the next stage, requested a stage ahead
    float hc[D], hh = 0.f;
    auto request = [&](int32_t k) {
        const int64_t at = hb + (k < k1 ? k : k0);
#pragma unroll
        for (int d = 0; d < D; ++d) hc[d] = g.c[d][at];
        hh = g.h[at];
    };
    // a hill past the range takes zero height on the first hill's centre
    auto factors = [&](int32_t i) {
        double(*f)[kTileHills][Ld] = s_f[i & 1];
        double L = k0 + i * kTileHills + wave < k1 ? (double)hh : 0.0, gd[D - 1], e, gl;
#pragma unroll
        for (int d = 0; d < D - 1; ++d) {
            axis_factor(g, d, xr[d], (double)hc[d], e, gd[d]);
            L *= e;
        }
        f[0][wave][lane] = L;
#pragma unroll
        for (int d = 0; d < D - 1; ++d) f[1 + d][wave][lane] = L * gd[d];
        axis_factor(g, D - 1, xc, (double)hc[D - 1], e, gl);
        f[D][wave][lane] = e;
        f[D + 1][wave][lane] = e * gl;
        request(k0 + (i + 1) * kTileHills + wave);
    };
    const int wr = wave >> 2, wc = wave & 3;
    const int32_t stages = (k1 - k0 + kTileHills - 1) / kTileHills;
    if (stages > 0) {
        request(k0 + wave);
        factors(0);
    }
    for (int32_t i = 0; i < stages; ++i) {
        __syncthreads();  // stage i's factors are written, stage i - 1's read
        if (i + 1 < stages) factors(i + 1);
        const double(*f)[kTileHills][Ld] = s_f[i & 1];
#pragma unroll
        for (int ks = 0; ks < kTileHills / 4; ++ks) {
            const int kk = 4 * ks + (lane >> 4), a = 16 * wr + (lane & 15), b = 16 * wc + (lane & 15);
            const double l0v = f[0][kk][a], e0 = f[D][kk][b];
            acc[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(l0v, e0, acc[0], 0, 0, 0);
#pragma unroll
            for (int d = 0; d < D - 1; ++d)
                acc[1 + d] = __builtin_amdgcn_mfma_f64_16x16x4f64(f[1 + d][kk][a], e0, acc[1 + d], 0, 0, 0);
            acc[D] = __builtin_amdgcn_mfma_f64_16x16x4f64(l0v, f[D + 1][kk][b], acc[D], 0, 0, 0);
        }
    }
    double *Vg, *Gg;
    node_sums<true>(g, l, slice, Vg, Gg);
    const int64_t c = c0 + 16 * wc + (lane & 15);
#pragma unroll
    for (int v = 0; v < 4; ++v) {
        const int64_t r = r0 + 16 * wr + (lane >> 4) + 4 * v;
        if (r >= nr || c >= nc) continue;
        const int64_t node = r * nc + c;
        Vg[node] = acc[0][v];
#pragma unroll
        for (int d = 0; d < D; ++d) Gg[(int64_t)d * g.N + node] = acc[1 + d][v];
    }
}

// Few hills (a list's own hill of a step, a short list): nothing to share
// over hills, so the nodes are shared out alone.  A workgroup takes 2^shift
// columns and as many rows as make four nodes a thread (one in one CV); a
// thread's nodes share their column's Gaussian, and the CVs of a row are one
// exponent.  One hill is a chain of its loads, one exponential and the nodes'
// update; each further one adds 0.6 us (0.2 in one CV).
constexpr int kFewRows = 4;  // nodes of a thread, D > 1

template <int D, bool REBUILD>
__global__ void __launch_bounds__(kBlock) k_grid_few(GridArgs g, int32_t l0, int32_t per, int32_t nr,
                                                     int32_t shift)
{
    constexpr int R = D == 1 ? 1 : kFewRows, DR = D == 1 ? 1 : D - 1;  // (one CV: no rows, DR unused)
    if (!REBUILD) advance_step(g);
    const int32_t l = REBUILD ? l0 : (int32_t)blockIdx.x / per, wg = (int32_t)blockIdx.x % per;
    int32_t k0, k1;
    hill_range<REBUILD>(g, l, 0, k0, k1);
    if (!REBUILD && k1 == k0) return;  // uniform
    const int64_t hb = (int64_t)g.wrec[l].hb4 * 4;
    const int32_t nc = g.n[D - 1];
    const int32_t side = 1 << shift, down = kBlock >> shift;  // columns of a tile, threads down it
    const int32_t tc = (nc + side - 1) >> shift, tiles = tc * ((nr + down * R - 1) / (down * R));
    double *const Vg = g.V + (int64_t)l * g.N, *const Gg = g.G + (int64_t)l * D * g.N;
    for (int32_t tile = wg; tile < tiles; tile += per) {
        const int32_t c = tile % tc * side + ((int32_t)threadIdx.x & (side - 1));
        const int32_t r0 = tile / tc * (down * R) + ((int32_t)threadIdx.x >> shift);
        const double xc = g.lo[D - 1] + (double)c * g.delta[D - 1];
        double xr[R][DR], acc[R][1 + D];
#pragma unroll
        for (int q = 0; q < R; ++q) {
            int32_t r = r0 + q * down;
#pragma unroll
            for (int d = D - 2; d >= 0; --d) {
                xr[q][d] = g.lo[d] + (double)(r % g.n[d]) * g.delta[d];
                r /= g.n[d];
            }
#pragma unroll
            for (int j = 0; j <= D; ++j) acc[q][j] = 0.0;
        }
        for (int32_t k = k0; k < k1; ++k) {
            double hc[D];
#pragma unroll
            for (int d = 0; d < D; ++d) hc[d] = (double)g.c[d][hb + k];
            double ec, gc;
            axis_factor(g, D - 1, xc, hc[D - 1], ec, gc);
            ec *= (double)g.h[hb + k];
#pragma unroll
            for (int q = 0; q < R; ++q) {
                double y = 0.0, gr[DR], yd;
#pragma unroll
                for (int d = 0; d < D - 1; ++d) {
                    gr[d] = -axis_offset(g, d, xr[q][d], hc[d], yd) * g.inv_sig2[d];
                    y += yd;
                }
                const double e = D == 1 ? ec : ec * exp2_neg(y);
                acc[q][0] += e;
#pragma unroll
                for (int d = 0; d < D - 1; ++d) acc[q][1 + d] = fma(e, gr[d], acc[q][1 + d]);
                acc[q][D] = fma(e, gc, acc[q][D]);
            }
        }
#pragma unroll
        for (int q = 0; q < R; ++q) {
            const int32_t r = r0 + q * down;
            if (r >= nr || c >= nc) continue;
            const int64_t node = (int64_t)r * nc + c;
            Vg[node] = REBUILD ? acc[q][0] : Vg[node] + acc[q][0];
#pragma unroll
            for (int d = 0; d < D; ++d) {
                double *p = Gg + (int64_t)d * g.N + node;
                *p = REBUILD ? acc[q][1 + d] : *p + acc[q][1 + d];
            }
        }
    }
    if (REBUILD) return;
    __syncthreads();  // every wavefront has read the count
    finish_add(g, l, k1, per);
}

// a rebuild's slices joined in order
__global__ void __launch_bounds__(kBlock) k_grid_join(GridArgs g, int32_t l)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x, n = (1 + g.D) * g.N;
    if (i >= n) return;
    double v = 0.0;
    int32_t s = 0;
    for (; s + 16 <= g.slices; s += 16) {  // 16 slices' sums in flight
        double p[16];
#pragma unroll
        for (int q = 0; q < 16; ++q) p[q] = g.part[(s + q) * n + i];
#pragma unroll
        for (int q = 0; q < 16; ++q) v += p[q];
    }
    for (; s < g.slices; ++s) v += g.part[s * n + i];
    if (i < g.N)
        g.V[(int64_t)l * g.N + i] = v;
    else
        g.G[(int64_t)l * g.D * g.N + i - g.N] = v;
}

int64_t tiles_of(int32_t D, const int32_t *n, int64_t N, int side)
{
    if (D == 1) return (N + 63) / 64;
    const int64_t nc = n[D - 1], nr = N / nc;
    return ((nc + side - 1) / side) * ((nr + side - 1) / side);
}

// 64 x 64 tiles where they cost less with their padding (three CVs' 12 to 32
// columns: 32 x 32) and are more than one, which kMostSlices parts do not
// spread over the chip (64 x 64 nodes 167 us, in 32 x 32 tiles 156).
bool fill_tiles(int32_t D, const int32_t *n, int64_t N)
{
    if (D == 1) return false;
    const int64_t large = tiles_of(D, n, N, kFillSide);
    return large > 1 && kFillCost * large < 10 * tiles_of(D, n, N, kTileSide);
}

template <bool REBUILD>
hipError_t launch_tiles(const GridArgs &g, int32_t l0, int64_t per, int64_t nz, hipStream_t s)
{
    constexpr int KG = REBUILD ? 4 : 1;
    if (per * nz > INT32_MAX) return hipErrorInvalidValue;
    const dim3 grid((unsigned)(per * nz));
    switch (g.D) {
    case 1: hipLaunchKernelGGL(k_grid_line<REBUILD>, grid, dim3(64 * kLineSlices), 0, s, g, l0, (int32_t)per); break;
    case 2: hipLaunchKernelGGL((k_grid_tiles<2, KG, REBUILD>), grid, dim3(256 * KG), 0, s, g, l0, (int32_t)per); break;
    case 3: hipLaunchKernelGGL((k_grid_tiles<3, KG, REBUILD>), grid, dim3(256 * KG), 0, s, g, l0, (int32_t)per); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// k_grid_few (the plan holds N to 2^30) on grids l0 .. l0 + nl - 1, at most `most` workgroups
// each: tiles of 64 columns, fewer where there are fewer, more where the rows
// would not fill them
template <bool REBUILD>
hipError_t launch_few(const GridArgs &g, int32_t l0, int64_t most, int64_t nl, hipStream_t s)
{
    const int32_t nc = g.n[g.D - 1], nr = (int32_t)(g.N / nc), rows = g.D == 1 ? 1 : kFewRows;
    int32_t shift = 0;
    while ((1 << shift) < nc && (shift < 6 || (shift < 8 && (kBlock >> (shift + 1)) * rows >= nr))) ++shift;
    if (g.D == 1) shift = 8;
    const int32_t side = 1 << shift, down = (kBlock >> shift) * rows;
    const int64_t per = std::min(most, (int64_t)((nc + side - 1) / side) * ((nr + down - 1) / down));
    if (per * nl > INT32_MAX) return hipErrorInvalidValue;
    const dim3 grid((unsigned)(per * nl));
    switch (g.D) {
    case 1: hipLaunchKernelGGL((k_grid_few<1, REBUILD>), grid, dim3(kBlock), 0, s, g, l0, (int32_t)per, nr, shift); break;
    case 2: hipLaunchKernelGGL((k_grid_few<2, REBUILD>), grid, dim3(kBlock), 0, s, g, l0, (int32_t)per, nr, shift); break;
    case 3: hipLaunchKernelGGL((k_grid_few<3, REBUILD>), grid, dim3(kBlock), 0, s, g, l0, (int32_t)per, nr, shift); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

__global__ void __launch_bounds__(kBlock) k_grid_eval(GridArgs g, int32_t l, const double *xi, int64_t n, double *V,
                                                        double *dV)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    double v, G[kMaxBiasDim];
    grid_read(g, l, xi + i * g.D, v, G);
    V[i] = v;
    if (dV)
        for (int d = 0; d < g.D; ++d) dV[i * g.D + d] = G[d];
}

__global__ void __launch_bounds__(kBlock) k_scale_f64(double *x, int64_t n, double a)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) x[i] *= a;
}

}  // namespace

hipError_t launch_scale_f64(double *x, int64_t n, double a, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_scale_f64, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, x, n, a);
    return hipGetLastError();
}

// Does k_grid_few take a step's hills?  One a list (private lists) always, one
// or two walkers of a shared list about even; in one CV up to 64 where the
// grid is more than one round of k_grid_line's workgroups.  A step that
// deposits, us with the tiles and with k_grid_few:
//   32 lists of 4,096 nodes in one CV          22.4  12.4
//   32 lists of 1,000 x 2 nodes                23.0  12.1
//   32 lists of 100 x 100 x 3                 136.2  30.9
//   a list of 512 x 512, 1 hill / 2 / 4        15.0  14.6 / 15.6  15.9 / 15.7  16.8
//   a list of 100,000 in one CV, 4 / 64        21.8  14.0 / 26.1  24.4
// A rebuild of up to 8 hills, 32 where padding is most of the tiles:
//   512 x 512, 4 hills / 16                    72.5  71.8 / 72.2  78.3
//   100 x 100 x 3, 16 / 64                    124.4  92.4 / 179   124
//   100,000 in one CV, 16 / 256                75.6  59.3 / 104   110
bool few_hills(const GridArgs &g, int64_t tiles)
{
    const int32_t hills = g.shared ? g.tabs.W : 1;
    return hills <= 2 || (g.D == 1 && tiles > 512 && hills <= 64);
}

bool few_rebuild(const GridArgs &g, int64_t hills)
{
    const int64_t tiles = tiles_of(g.D, g.n, g.N, kTileSide);
    if (g.D == 1) return hills <= (tiles > 512 ? 64 : 8);
    return hills <= (tiles * kTileSide * kTileSide >= 4 * g.N ? 32 : 8);
}

// A configuration that never deposits (deposit off, or on a stride of 0)
// has nothing for the add kernel but the step counter: the step kernel then
// advances it and the add kernel is not launched.
hipError_t launch_grid_step(const GridArgs &g0, hipStream_t s)
{
    GridArgs g = g0;
    const bool add = !(g.deposit == 0 || (g.deposit == 1 && g.stride <= 0));
    g.count_in_step = add ? 0 : g.count_step;
    if (g.tabs.W < 1 || g.L < 1) return hipErrorInvalidValue;
    const bool wave = g.do_forces && g.small.on && g.small.U > 0;
    if (g.fuse_cv && !wave) return hipErrorInvalidValue;  // only the wavefront step evaluates CVs
    if (wave)
        hipLaunchKernelGGL(k_grid_step_wave, dim3(g.tabs.W), dim3(64), 0, s, g);
    else
        hipLaunchKernelGGL(k_grid_step, dim3(g.tabs.W), dim3(kBlock), 0, s, g);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || !add) return e;
    // about 1024 workgroups in all (512 of k_grid_line's 16 wavefronts): on a
    // step that deposits nothing each of them only reads its list's count of
    // new hills
    const int64_t tiles = tiles_of(g.D, g.n, g.N, kTileSide), room = g.D == 1 ? 512 : 1024;
    const int64_t most = (room + g.L - 1) / g.L;
    if (few_hills(g, tiles)) return launch_few<false>(g, 0, (1024 + g.L - 1) / g.L, g.L, s);
    return launch_tiles<false>(g, 0, std::min(tiles, most), g.L, s);
}

// A workgroup fills a compute unit, so the tiles of most grids leave the chip
// idle or a last round of it nearly empty: the list is summed in `slices`
// parts, as many as give the fewest rounds per part, at most four
// rounds.  Records of (1 + D) N sums a slice, joined in order.  30,000
// hills, upload included: 100 x 100 nodes 1,499 us unsliced in
// 32 x 32 tiles, 147 now; 24 x 24 x 24 2,427 and 249; 512 x 512 1,057 now.
int32_t grid_slices(int32_t D, const int32_t *n, int64_t N)
{
    const int64_t tiles = tiles_of(D, n, N, fill_tiles(D, n, N) ? kFillSide : kTileSide);
    const int64_t at_once = D == 1 ? 512 : 256;  // one CV's sums: two workgroups a compute unit
    int32_t best = 1;
    for (int32_t s = 2; s <= kMostSlices && s * tiles <= 4 * at_once; ++s)
        if ((s * tiles + at_once - 1) / at_once * best < (best * tiles + at_once - 1) / at_once * s) best = s;
    return best;
}

hipError_t launch_grid_rebuild(const GridArgs &g0, int32_t l, int64_t hills, hipStream_t s)
{
    GridArgs g = g0;
    if (l < 0 || l >= g.L || g.slices < 1 || (g.slices > 1 && !g.part)) return hipErrorInvalidValue;
    if (few_rebuild(g, hills)) {
        g.slices = 1;
        return launch_few<true>(g, l, 4096, 1, s);
    }
    g.slices = (int32_t)std::min<int64_t>(g.slices, (hills + kTileHills - 1) / kTileHills);  // none of them empty
    hipError_t e;
    if (fill_tiles(g.D, g.n, g.N)) {
        const int64_t tiles = tiles_of(g.D, g.n, g.N, kFillSide);
        if (tiles * g.slices > INT32_MAX) return hipErrorInvalidValue;
        const dim3 grid((unsigned)(tiles * g.slices));
        if (g.D == 2)
            hipLaunchKernelGGL(k_grid_fill<2>, grid, dim3(1024), 0, s, g, l, (int32_t)tiles);
        else
            hipLaunchKernelGGL(k_grid_fill<3>, grid, dim3(1024), 0, s, g, l, (int32_t)tiles);
        e = hipGetLastError();
    } else {
        e = launch_tiles<true>(g, l, std::min<int64_t>(tiles_of(g.D, g.n, g.N, kTileSide), 4096), g.slices, s);
    }
    if (e != hipSuccess || g.slices == 1) return e;
    const int64_t n = (1 + g.D) * g.N;
    hipLaunchKernelGGL(k_grid_join, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, g, l);
    return hipGetLastError();
}

hipError_t launch_grid_eval(const GridArgs &g, int32_t l, const double *xi, int64_t n, double *V, double *dV,
                            hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    if (l < 0 || l >= g.L) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_grid_eval, dim3((unsigned)((n + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, g, l, xi, n, V,
                       dV);
    return hipGetLastError();
}

}  // namespace sx
