// Hill sum over ONE hill list shared by many query points (walkers sharing
// a bias, or arbitrary evaluation points such as training and
// certification samples of a surrogate).  Metadynamics bias, Sec. 2.1.5.
//
// Unlike the private-list sum, every hill is reused by every query, so the
// work is bound by VALU arithmetic, not by HBM:
//   * grid x: hill chunks, an equal share of the hills in the list each
//     (formed from the count on the device, so a list with spare capacity
//     keeps every workgroup busy); grid y: blocks of ql Q queries;
//   * the four wavefronts of a workgroup hold the same queries (Q per lane)
//     and split every staged group of 256 hills in four; with fewer than 64
//     queries, ql = 32, 16, 8 or 4 lanes hold them and the 64 / ql lane groups
//     split the wavefront's hills (32 queries on 64 lanes left half of them
//     idle); shuffles and a fixed-order LDS reduction join all of them;
//   * staging converts each hill once to FP64: a periodic CV in turns less
//     one half, so that f = fract(xi - c + 1/2) is the minimum image plus one
//     half in two operations, and w f (f - 1) + w / 4 its term of the
//     quadratic form in two more; another CV scaled by
//     sqrt(log2(e) / (2 sigma^2)).  With the Gaussian (one v_exp_f32, half
//     rate) and FP64 sums of e and e f, a (hill, query) pair of two periodic
//     CVs takes 16 issue slots (18 with a scaled displacement and
//     x - P rint(x / P)).  The sum of e (f - 1/2) is formed once per chunk.
//     Summing the products in FP32 would lose digits where the terms of
//     dV/dxi cancel;
//   * which CVs are periodic is a template parameter, a bit per CV (8,191
//     points on 200,000 hills, an angle and a distance: 680 us; with a test of
//     the period in the pair loop 1,149);
//   * when every CV is a dihedral a step's workgroups evaluate their queries'
//     CVs themselves (FP64) while their first hills are in flight, which
//     saves the CV kernel's launch; the first chunk's workgroups store xi and
//     the Jacobian for the finalize;
//   * each (chunk, query) partial has one writer; the finalize kernel sums a
//     query's chunks in chunk order (bitwise deterministic), forms dV/dxi,
//     and appends one hill per walker for a deposition step, in walker order;
//     the last of its workgroups to arrive then moves the count.
// A step of 256 walkers on 100,000 hills: 22.7 us (34.7 with a CV launch, a
// count launch, 18 slots per pair and 784 unequal workgroups); 131,072 points
// on 100,000 hills: 5.45 ms = 2.4 x 10^12 pairs/s, the 38 T issue slots/s that
// a loop of multiply-adds reaches (6.24 ms).
#include "sx_internal.h"
#include "dev_cv.h"
#include "dev_reduce.h"
#include "dev_gather.h"

namespace sx {
namespace {

constexpr int kStage = kBlock;  // hills staged in LDS at a time (one per lane)
constexpr int64_t kMaxRecords = 8 * 65536;  // partial records of a sum at arbitrary points

// Periodic CVs of a shared sum: bit d for CV d, or kNarrowForm where one of
// them is narrower than kNarrow; of the fallback sums, one of the three.
constexpr int kNarrowForm = -1;
constexpr int all_periodic(int D) { return (1 << D) - 1; }
enum { kPerNone = 0, kPerAll = 1, kPerMixed = 2 };

// The exponent as w f (f - 1) + w / 4 cancels near a hill's centre: its error
// is that of w / 4, 7.1 / sigma^2, in FP64, about 1e-14 / sigma^2 for three
// CVs.  Narrower than kNarrow that would pass 2^-31 (the Gaussian's own float32
// rounding is 2^-24; at 1e-5 rad sums came out up to 1.4e-5 off), so such sums
// keep the square of a displacement in units of the width, two issue slots more.
constexpr double kNarrow = 0.005;

int periodic_form(const SharedArgs &a)
{
    int m = 0;
    for (int d = 0; d < a.D; ++d)
        if (a.period[d] > 0.0) {
            if (a.inv_sig2[d] * (kNarrow * kNarrow) > 1.0) return kNarrowForm;
            m |= 1 << d;
        }
    return m;
}

// Queries per lane (Q) and lanes that hold queries (ql) of a sum over nq
// queries of a list with room for cap hills.  More queries per lane amortise
// the staged hills' LDS reads, but a lane's queries are one chain: their start
// and their sums at the end are paid by fewer wavefronts.  So Q rises with the
// pairs a launch has (by the capacity: the count is on the device).  Two
// angles, us with Q = 1, 2, 4:
//     1,000 hills x  8,192 points   11.1  11.5  14.9
//    10,000 hills x  4,096          27.5  28.8  29.6
//    10,000 hills x 16,384          84.5  80.6  81.8
//   100,000 hills x  1,024          56.3  54.0  56.2
//    30,000 hills x 16,384         241.2 224.3 220.2
//   100,000 hills x 16,384         784.2 729.1 712.5
// and a list with spare capacity (1,000 hills in room for 300,000) pays up to
// 1.3 times its best at 1,024 points.  More than 65,536 queries are walkers:
// 4, so that their blocks fit a grid.
void shared_shape(int64_t nq, int64_t cap, int &Q, int &ql)
{
    const double pairs = (double)cap * (double)nq;
    Q = nq > 65536 || (nq >= 8192 && pairs >= 0x1p29) ? 4 : nq >= 1024 && pairs >= 0x1p26 ? 2 : 1;
    ql = 64;
    while (ql > 4 && nq <= ql / 2) ql /= 2;
}

// Dihedral d of the walker whose atoms start at aoff (T: the position type);
// the atom indices and slot are selected by value from the kernel arguments.
template <int D, typename T>
__device__ __forceinline__ double query_dihedral(const CvSet &cs, const PosView &pos, int64_t aoff, int d, double3 (&g)[4],
                                                 int32_t &slot0)
{
    int32_t at[4];
    slot0 = cs.cv[0].slot0;
#pragma unroll
    for (int q = 0; q < 4; ++q) at[q] = cs.cv[0].atom[q];
#pragma unroll
    for (int dd = 1; dd < D; ++dd) {
        slot0 = d == dd ? cs.cv[dd].slot0 : slot0;
#pragma unroll
        for (int q = 0; q < 4; ++q) at[q] = d == dd ? cs.cv[dd].atom[q] : at[q];
    }
    double3 r[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) r[q] = ld_pos_t<T>(pos, aoff + at[q]);
    return dihedral_fp64<true>(r, g);
}

template <int D, int Q, int PER, bool FUSE>
__device__ __forceinline__ void hill_shared(const SharedArgs &a, const SharedCv *fc)
{
    __shared__ double s_c[kStage][D];
    __shared__ float s_h[kStage];
    __shared__ double s_red[3][Q * (1 + D)][64];
    __shared__ double s_xi[FUSE ? D : 1][FUSE ? 64 * Q : 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // the step counter moves here (the finalize, which may deposit, reads it)
    if (a.count_step && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0)
        *a.dstep = a.step >= 0 ? a.step + 1 : *a.dstep + 1;
    const int32_t n = *a.count;
    // ql lanes hold queries; G = 64 / ql = 2^lg groups of them split the hills
    const int lg = Q > 1 ? 0 : a.lg, ql = 64 >> lg, G = 1 << lg;
    const int qlane = lane & (ql - 1), grp = lane >> (6 - lg);
    const int64_t qb0 = (int64_t)blockIdx.y * ql * Q;
    const int64_t nq = a.nq;
    // this workgroup's share of the hills
    const int64_t share = (((int64_t)n + a.nchunk - 1) / a.nchunk + 3) / 4 * 4;
    const int64_t h0 = min((int64_t)n, (int64_t)blockIdx.x * share), hend = min((int64_t)n, h0 + share);
    // the first stage's hills, requested ahead of the CVs
    float cn[D], hn = 0.f;
    auto request = [&](int64_t k) {
        const bool ok = k < hend;
#pragma unroll
        for (int d = 0; d < D; ++d) cn[d] = ok ? a.c[d][k] : 0.f;
        hn = ok ? a.h[k] : 0.f;  // zero height: no contribution
    };
    request(h0 + threadIdx.x);
    if (FUSE) {
        for (int it = threadIdx.x; it < ql * Q * D; it += kBlock) {
            const int d = it / (ql * Q), i = it % (ql * Q);
            const int64_t w = qb0 + i;
            if (w >= nq) continue;
            const int64_t aoff = a.tabs.atom_off[w];
            double3 g[4];
            int32_t slot0;
            const double x = fc->pos.f64 ? query_dihedral<D, double>(fc->cs, fc->pos, aoff, d, g, slot0)
                                         : query_dihedral<D, float>(fc->cs, fc->pos, aoff, d, g, slot0);
            s_xi[d][i] = x;
            if (blockIdx.x == 0) {
                fc->xi_ws[w * D + d] = x;
                float *js = fc->J_ws + (w * a.nslots + slot0) * 3;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    js[3 * q] = (float)g[q].x;
                    js[3 * q + 1] = (float)g[q].y;
                    js[3 * q + 2] = (float)g[q].z;
                }
            }
        }
        __syncthreads();
    }
    // scale of CV d: turns (periodic), or units in which the quadratic form
    // is the square; wt: the periodic CV's weight of f (f - 1) + 1/4
    constexpr double kInvTurn = 0.15915494309189533577, kTurn = 6.2831853071795864769;
    // (kNarrowForm: all of them scaled, and the periods with them)
    constexpr bool kScaled = PER == kNarrowForm;
    double sc[D], wt[D], per[D], iper[D], q0 = 0.0;
    bool wrap[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        const double s2 = 0.72134752044448170368 * a.inv_sig2[d];  // log2(e) / (2 sigma^2)
        wrap[d] = !kScaled && (PER >> d & 1);
        wt[d] = wrap[d] ? s2 * (kTurn * kTurn) : 0.0;
        sc[d] = wrap[d] ? kInvTurn : sqrt(s2);
        per[d] = kScaled ? a.period[d] * sc[d] : 0.0;
        iper[d] = kScaled ? a.inv_period[d] / sc[d] : 0.0;
        q0 += 0.25 * wt[d];
    }
    double xs[Q][D];
    bool live[Q];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        const int64_t q = qb0 + qlane + (int64_t)ql * i;
        live[i] = q < nq;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            const double x = !live[i] ? 0.0 : FUSE ? s_xi[FUSE ? d : 0][FUSE ? qlane + ql * i : 0] : a.xi[q * D + d];
            xs[i][d] = x * sc[d];
        }
    }
    double acc[Q][1 + D];
#pragma unroll
    for (int i = 0; i < Q; ++i)
#pragma unroll
        for (int j = 0; j <= D; ++j) acc[i][j] = 0.0;
    for (int64_t s0 = h0; s0 < hend; s0 += kStage) {
#pragma unroll
        for (int d = 0; d < D; ++d)
            s_c[threadIdx.x][d] = wrap[d] ? fma((double)cn[d], sc[d], -0.5) : (double)cn[d] * sc[d];
        s_h[threadIdx.x] = hn;
        __syncthreads();
        request(s0 + kStage + threadIdx.x);
        // this wavefront's quarter of the staged hills in steps of 4 G, four
        // neighbours per lane group (4 G <= 64, so at most 64 a wavefront)
        const int m = (int)min((int64_t)kStage, hend - s0);
        const int steps = ((m + 3) / 4 + 4 * G - 1) >> (2 + lg);
        int jb = wave * steps * 4 * G + 4 * grp;
        for (int st = 0; st < steps; ++st, jb += 4 * G) {
#pragma unroll
            for (int u = 0; u < 4; ++u) {  // past m: zero height
                const int j = jb + u;
                double c[D];
#pragma unroll
                for (int d = 0; d < D; ++d) c[d] = s_c[j][d];
                const float h = s_h[j];
#pragma unroll
                for (int i = 0; i < Q; ++i) {
                    double x[D], qd = q0;
#pragma unroll
                    for (int d = 0; d < D; ++d) {
                        x[d] = xs[i][d] - c[d];
                        if (wrap[d]) {
                            x[d] = __builtin_amdgcn_fract(x[d]);
                            qd = fma(x[d], fma(wt[d], x[d], -wt[d]), qd);
                        } else {
                            if (kScaled && per[d] > 0.0) x[d] = fma(-per[d], rint(x[d] * iper[d]), x[d]);
                            qd = fma(x[d], x[d], qd);
                        }
                    }
                    const double e = (double)(h * __builtin_amdgcn_exp2f(-(float)qd));
                    acc[i][0] += e;
#pragma unroll
                    for (int d = 0; d < D; ++d) acc[i][1 + d] = fma(e, x[d], acc[i][1 + d]);
                }
            }
        }
        __syncthreads();
    }
    // join the lane groups, then the four wavefronts in a fixed order (0 + 1 + 2 + 3)
    if (Q == 1)
        for (int o = ql; o < 64; o <<= 1)
#pragma unroll
            for (int j = 0; j <= D; ++j) acc[0][j] += __shfl_xor(acc[0][j], o, 64);
    if (wave > 0) {
#pragma unroll
        for (int i = 0; i < Q; ++i)
#pragma unroll
            for (int j = 0; j <= D; ++j) s_red[wave - 1][i * (1 + D) + j][lane] = acc[i][j];
    }
    __syncthreads();
    if (wave != 0 || grp != 0) return;
#pragma unroll
    for (int w = 0; w < 3; ++w)
#pragma unroll
        for (int i = 0; i < Q; ++i)
#pragma unroll
            for (int j = 0; j <= D; ++j) acc[i][j] += s_red[w][i * (1 + D) + j][lane];
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        if (!live[i]) continue;
        const int64_t q = qb0 + qlane + (int64_t)ql * i;
        double *p = a.partial + ((int64_t)blockIdx.x * a.rec_ch + q * a.rec_q) * 4;
        p[0] = acc[i][0];
#pragma unroll
        for (int d = 0; d < D; ++d)  // back to CV units
            p[1 + d] = wrap[d] ? kTurn * (acc[i][1 + d] - 0.5 * acc[i][0]) : acc[i][1 + d] / sc[d];
    }
}

template <int D, int Q, int PER>
__global__ void __launch_bounds__(kBlock) k_hill_shared(SharedArgs a)
{
    hill_shared<D, Q, PER, false>(a, nullptr);
}

template <int D, int Q>
__global__ void __launch_bounds__(kBlock) k_hill_shared_cv(SharedArgs a, SharedCv fc)
{
    hill_shared<D, Q, all_periodic(D), true>(a, &fc);
}

// does this launch append hills?  (the step counter was moved by the sum)
__device__ __forceinline__ bool deposits(const SharedArgs &a)
{
    return a.deposit == 2 || (a.deposit == 1 && a.stride > 0 && (*a.dstep - 1) % a.stride == 0);
}

// The count of a shared list moves by the walkers' hills when the last
// workgroup of a depositing finalize arrives: by one thread per workgroup,
// after the workgroup's threads have read the count (a barrier, or one
// wavefront).  The ticket orders nothing else: the appended hills are read by
// later launches.  (A kernel of its own for this took 3.4 us on every step.)
__device__ __forceinline__ void shared_count(const SharedArgs &a, int32_t cnt)
{
    if (atomicAdd(a.tick, 1) != (int32_t)gridDim.x - 1) return;
    *a.tick = 0;
    if ((int64_t)cnt + a.nq <= a.cap) *a.count = (int32_t)(cnt + a.nq);
}

// per query: V, dV/dxi, outputs and (all or none) the appended hill;
// w is the query's row (its walker, or its evaluation point)
template <int D>
__device__ __forceinline__ void shared_finish(const SharedArgs &a, int64_t w, const double (&acc)[1 + D],
                                              double (&dv)[D])
{
    const double V = acc[0];
    bool finite = isfinite(V);
    if (a.V_ws) a.V_ws[w] = V;
    if (a.V_out) a.V_out[w] = V;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        dv[d] = -acc[1 + d] * a.inv_sig2[d];
        finite = finite && isfinite(dv[d]);
        if (a.dV_ws) a.dV_ws[w * D + d] = dv[d];
        if (a.dV_out) a.dV_out[w * D + d] = dv[d];
        if (a.xi_out) a.xi_out[w * D + d] = a.xi[w * D + d];
    }
    if (!finite && a.flags) atomicOr(a.flags, kFlagNonFinite);
    if (deposits(a)) {
        // all walkers append in walker order at count + w (all or none);
        // the count moves once every workgroup has read it
        const int32_t n = *a.count;
        if ((int64_t)n + a.nq <= a.cap) {
            const int64_t k = (int64_t)n + w;
#pragma unroll
            for (int d = 0; d < D; ++d) a.c[d][k] = (float)a.xi[w * D + d];
            a.h[k] = (float)(a.inv_kdT > 0.0 ? a.height * exp(-V * a.inv_kdT) : a.height);
        } else if (w == 0) {
            atomicOr(a.flags, kFlagCapacity);
        }
    }
}

// few chunks: one lane per query sums its chunks in order (no fallback mode)
template <int D>
__global__ void __launch_bounds__(kBlock) k_hill_shared_finalize(SharedArgs a)
{
    const int64_t q = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (q < a.nq) {
        double acc[1 + D];
#pragma unroll
        for (int j = 0; j <= D; ++j) acc[j] = 0.0;
#pragma unroll 4
        for (int ch = 0; ch < a.nchunk; ++ch) {
            const double *p = a.partial + ((int64_t)ch * a.rec_ch + q * a.rec_q) * 4;
#pragma unroll
            for (int j = 0; j <= D; ++j) acc[j] += p[j];
        }
        double dv[D];
        shared_finish<D>(a, q, acc, dv);
        if (a.do_forces) {  // coefficients -dV/dxi; this lane owns the walker's atoms
            double coef[D];
#pragma unroll
            for (int d = 0; d < D; ++d) coef[d] = -dv[d];
            const float *Jw = a.J + q * a.nslots * 3;
            for (int u = 0; u < a.tabs.U; ++u) gather_atom(a.tabs, Jw, (int32_t)q, coef, a.F, u);
        }
    }
    if (!deposits(a)) return;  // uniform
    const int32_t cnt = *a.count;
    __syncthreads();
    if (threadIdx.x == 0) shared_count(a, cnt);
}

// many chunks, or fallback sums: one workgroup per query (walker), lanes
// stride over the chunks and a fixed reduction tree combines them
// (deterministic); then the walker's force gather
template <int D>
__global__ void __launch_bounds__(kBlock) k_hill_shared_finalize_wg(SharedArgs a)
{
    __shared__ double lds[(1 + D) * (kBlock / 64)];
    __shared__ double s_coef[D];
    const int64_t w = blockIdx.x, q = w;  // fallback mode: records per walker
    if (a.fb && !a.fb[w]) return;           // uniform per workgroup
    double acc[1 + D];
#pragma unroll
    for (int j = 0; j <= D; ++j) acc[j] = 0.0;
    for (int ch = threadIdx.x; ch < a.nchunk; ch += kBlock) {
        const double *p = a.partial + ((int64_t)ch * a.rec_ch + q * a.rec_q) * 4;
#pragma unroll
        for (int j = 0; j <= D; ++j) acc[j] += p[j];
    }
    block_sum0<1 + D>(acc, lds);
    if (threadIdx.x == 0) {
        double dv[D];
        shared_finish<D>(a, w, acc, dv);
#pragma unroll
        for (int d = 0; d < D; ++d) s_coef[d] = -dv[d];
        if (deposits(a)) shared_count(a, *a.count);  // this thread alone reads the count
    }
    if (!a.do_forces) return;  // uniform
    __syncthreads();
    gather_forces(a.tabs, a.J + w * a.nslots * 3, (int32_t)w, s_coef, a.F);
}

// The same in one wavefront, for steps that gather forces through the
// table in kernel-argument form: every load is requested before the first
// wait (each lane's first four chunk records -- lanes past the count re-read
// the last one and drop it, nchunk >= 1 -- the CV values, the deposit's count
// and step, and a table row per lane with its Jacobian rows and force; lanes
// past U re-read row U - 1 and store nothing); the records are summed
// lane-strided and combined by a butterfly (every lane ends with the same
// bits); lane 0 writes the outputs and deposits, lane u < U adds atom u's
// force.  No LDS, no barrier.
template <int D>
__global__ void __launch_bounds__(64) k_hill_shared_finalize_wave(SharedArgs a)
{
    const int64_t w = blockIdx.x, q = w;  // fallback mode: records per walker
    const int lane = threadIdx.x;
    if (a.fb && !a.fb[w]) return;  // uniform per workgroup
    const int nch = a.nchunk;
    constexpr int RB = 4;  // records of a lane in flight
    double r0[RB][1 + D];
#pragma unroll
    for (int b = 0; b < RB; ++b) {
        const double *p = a.partial + ((int64_t)min(lane + 64 * b, nch - 1) * a.rec_ch + q * a.rec_q) * 4;
#pragma unroll
        for (int j = 0; j <= D; ++j) r0[b][j] = p[j];
    }
    double xi[D];
#pragma unroll
    for (int d = 0; d < D; ++d) xi[d] = a.xi[w * D + d];
    const bool dep_cnt = a.deposit == 1 && a.stride > 0;
    const int64_t dstep = dep_cnt ? *a.dstep : 0;
    const int32_t cnt = a.deposit ? *a.count : 0;
    SmallGather sg{0.f, 0.f, 0.f, nullptr};
    int nent = 0;
    int32_t ent[kSmallPer];
    float jr[kSmallPer][3];
    small_rows(a.small, a.J + w * a.nslots * 3, a.F, a.tabs.atom_off[w], min(lane, a.small.U - 1), sg, nent, ent, jr);
    // the first records kept or replaced by +0.0 through a bit mask, which
    // uses the loaded value on every lane (a select lets the load move
    // under a branch)
    double acc[1 + D];
#pragma unroll
    for (int j = 0; j <= D; ++j) acc[j] = 0.0;
#pragma unroll
    for (int b = 0; b < RB; ++b) {
        const long long keep = lane + 64 * b < nch ? -1LL : 0LL;
#pragma unroll
        for (int j = 0; j <= D; ++j) acc[j] += __longlong_as_double(__double_as_longlong(r0[b][j]) & keep);
    }
#pragma unroll 4
    for (int ch = lane + 64 * RB; ch < nch; ch += 64) {  // the same order as one loop from ch = lane
        const double *p = a.partial + ((int64_t)ch * a.rec_ch + q * a.rec_q) * 4;
#pragma unroll
        for (int j = 0; j <= D; ++j) acc[j] += p[j];
    }
#pragma unroll
    for (int j = 0; j <= D; ++j) acc[j] = wave_sum(acc[j]);
    double dv[D];
#pragma unroll
    for (int d = 0; d < D; ++d) dv[d] = -acc[1 + d] * a.inv_sig2[d];
    // ahead of lane 0's outputs, whose arithmetic then overlaps these stores
    if (lane < a.small.U) {
        double coef[D];
#pragma unroll
        for (int d = 0; d < D; ++d) coef[d] = -dv[d];
        small_forces(a.small, a.F, sg, nent, ent, jr, coef);
    }
    if (lane == 0) {
        const double V = acc[0];
        bool finite = isfinite(V);
        if (a.V_ws) a.V_ws[w] = V;
        if (a.V_out) a.V_out[w] = V;
#pragma unroll
        for (int d = 0; d < D; ++d) {
            finite = finite && isfinite(dv[d]);
            if (a.dV_ws) a.dV_ws[w * D + d] = dv[d];
            if (a.dV_out) a.dV_out[w * D + d] = dv[d];
            if (a.xi_out) a.xi_out[w * D + d] = xi[d];
        }
        if (!finite && a.flags) atomicOr(a.flags, kFlagNonFinite);
        bool dep = a.deposit == 2;
        if (dep_cnt) dep = (dstep - 1) % a.stride == 0;
        if (dep) {  // as shared_finish: walker order at count + w, all or none
            if ((int64_t)cnt + a.nq <= a.cap) {
                const int64_t k = (int64_t)cnt + w;
#pragma unroll
                for (int d = 0; d < D; ++d) a.c[d][k] = (float)xi[d];
                a.h[k] = (float)(a.inv_kdT > 0.0 ? a.height * exp(-V * a.inv_kdT) : a.height);
            } else if (w == 0) {
                atomicOr(a.flags, kFlagCapacity);
            }
            shared_count(a, cnt);
        }
    }
}

// Fallback sums of a surrogate step (the few walkers outside certified
// cells): workgroup (c, y) sums chunk c of kQmChunk hills for its walkers,
// lanes over hills with float4 loads all issued before use (the chunk is
// read from L2 once per workgroup and kept in registers for all of its
// walkers), a fixed-order reduction, one partial record per (chunk,
// walker); the finalize kernel then sums a walker's chunks in order.
// COMPACT (at most kQmCompactMax queries): gridDim.y = min(queries,
// kQmSlots) rows, row y taking the flagged walkers of rank y, y + rows, ...
// in walker order, so the grid does not grow with the walkers the network
// serves; otherwise row y is walker y and leaves at once unless flagged.
// A walker's records do not depend on which workgroup formed them.
constexpr int kQmChunk = 4096;               // hills per workgroup
constexpr int kQmGroups = kQmChunk / (4 * kBlock);  // float4 groups per lane
constexpr int kQmSlots = 32;                 // workgroup rows of the compacted grid
constexpr int kQmCompactMax = 1024;          // largest query count it serves
constexpr int kQmPerRow = kQmCompactMax / kQmSlots;  // walkers one row takes at most

template <int D, int PER, bool COMPACT>
__global__ void __launch_bounds__(kBlock) k_hill_shared_qm(SharedArgs a)
{
    __shared__ double lds[(1 + D) * (kBlock / 64)];
    __shared__ int32_t s_list[COMPACT ? kQmPerRow : 1];
    __shared__ int32_t s_nw;
    if (a.count_step && blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0)
        *a.dstep = a.step >= 0 ? a.step + 1 : *a.dstep + 1;
    int nw = 1;
    if (COMPACT) {
        // wavefront 0 ranks the flagged walkers in order and lists this row's
        if (threadIdx.x < 64) {
            const int lane = threadIdx.x;
            const unsigned long long below = (1ull << lane) - 1ull;
            int base = 0, mine = 0;
            for (int64_t b0 = 0; b0 < a.nq; b0 += 64) {
                const int64_t ww = b0 + lane;
                const bool f = ww < a.nq && a.fb[ww];
                const unsigned long long m = __ballot(f);
                const bool take = f && (base + __popcll(m & below)) % (int)gridDim.y == (int)blockIdx.y;
                const unsigned long long mt = __ballot(take);
                if (take) s_list[mine + __popcll(mt & below)] = (int32_t)ww;  // < kQmPerRow: at most nq / rows
                mine += __popcll(mt);
                base += __popcll(m);
            }
            if (lane == 0) s_nw = mine;
        }
        __syncthreads();
        nw = s_nw;
    } else if (!a.fb[blockIdx.y]) {
        return;  // uniform per workgroup
    }
    if (nw == 0) return;  // uniform
    const int32_t n = *a.count;
    const int64_t h0 = (int64_t)blockIdx.x * kQmChunk;
    if (h0 >= n) {  // uniform: a chunk past the count adds zero (the finalize sums every chunk)
        for (int iw = 0; iw < nw; ++iw) {
            const int64_t w = COMPACT ? (int64_t)s_list[iw] : (int64_t)blockIdx.y;
            if (threadIdx.x <= D) a.partial[((int64_t)blockIdx.x * a.nq + w) * 4 + threadIdx.x] = 0.0;
        }
        return;
    }
    double sc[D], per[D], iper[D];
    bool wrap[D];
#pragma unroll
    for (int d = 0; d < D; ++d) {
        sc[d] = sqrt(0.7213475204444817 * a.inv_sig2[d]);
        wrap[d] = PER == kPerAll || (PER == kPerMixed && a.period[d] > 0.0);
        per[d] = a.period[d] * sc[d];
        iper[d] = a.inv_period[d] / sc[d];
    }
    // groups of 4 hills; the list's storage is padded to a multiple of 4
    // floats and 16-byte aligned: a group past the count reads group 0 and
    // gets zero heights
    float4 cv[kQmGroups][D], hv[kQmGroups];
    int64_t kk[kQmGroups];
#pragma unroll
    for (int it = 0; it < kQmGroups; ++it) {
        const int64_t k = h0 + 4 * ((int64_t)it * kBlock + threadIdx.x);
        kk[it] = k;
        const int64_t ks = k < n ? k : 0;
#pragma unroll
        for (int d = 0; d < D; ++d) cv[it][d] = *reinterpret_cast<const float4 *>(a.c[d] + ks);
        hv[it] = *reinterpret_cast<const float4 *>(a.h + ks);
    }
    for (int iw = 0; iw < nw; ++iw) {
        const int64_t w = COMPACT ? (int64_t)s_list[iw] : (int64_t)blockIdx.y;
        double xs[D];
#pragma unroll
        for (int d = 0; d < D; ++d) xs[d] = a.xi[w * D + d] * sc[d];
        double acc[1 + D];
#pragma unroll
        for (int j = 0; j <= D; ++j) acc[j] = 0.0;
#pragma unroll
        for (int it = 0; it < kQmGroups; ++it) {
            const int64_t k = kk[it];
            const float hh[4] = {k < n ? hv[it].x : 0.f, k + 1 < n ? hv[it].y : 0.f, k + 2 < n ? hv[it].z : 0.f,
                                 k + 3 < n ? hv[it].w : 0.f};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                double x[D], qd = 0.0;
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    const float4 &c4 = cv[it][d];
                    const float c = j == 0 ? c4.x : (j == 1 ? c4.y : (j == 2 ? c4.z : c4.w));
                    x[d] = xs[d] - (double)c * sc[d];
                    if (wrap[d]) x[d] = fma(-per[d], rint(x[d] * iper[d]), x[d]);
                    qd = fma(x[d], x[d], qd);
                }
                const double e = (double)(hh[j] * __builtin_amdgcn_exp2f(-(float)qd));
                acc[0] += e;
#pragma unroll
                for (int d = 0; d < D; ++d) acc[1 + d] = fma(e, x[d], acc[1 + d]);
            }
        }
        block_sum0<1 + D>(acc, lds);  // ends with a barrier: lds is free for the next walker
        if (threadIdx.x == 0) {
            double *p = a.partial + ((int64_t)blockIdx.x * a.nq + w) * 4;
            p[0] = acc[0];
#pragma unroll
            for (int d = 0; d < D; ++d) p[1 + d] = acc[1 + d] / sc[d];  // back to CV units
        }
    }
}

// the one-wavefront finalize: forces through the kernel-argument table of
// walkers (one query per walker, its records at query w)
bool small_finalize(const SharedArgs &a)
{
    return a.do_forces && a.small.on && a.small.U > 0 && a.nchunk >= 1 && a.tabs.W == a.nq;
}

template <int D, int Q, int PER = kNarrowForm>
void launch_sum(const SharedArgs &a, const SharedCv *cv, dim3 grid, hipStream_t s)
{
    if (cv)
        hipLaunchKernelGGL((k_hill_shared_cv<D, Q>), grid, dim3(kBlock), 0, s, a, *cv);
    else if (periodic_form(a) == PER)
        hipLaunchKernelGGL((k_hill_shared<D, Q, PER>), grid, dim3(kBlock), 0, s, a);
    else if constexpr (PER < all_periodic(D))
        launch_sum<D, Q, PER + 1>(a, cv, grid, s);
}

template <int D>
hipError_t launch_shared_d(const SharedArgs &a, const SharedCv *cv, hipStream_t s)
{
    if (a.fb) {  // fallback walkers of a surrogate step: query-major sums, finalize per walker
        SharedArgs b = a;
        b.nchunk = (int32_t)std::max<int64_t>(1, (a.cap + kQmChunk - 1) / kQmChunk);
        b.rec_ch = a.nq;
        b.rec_q = 1;
        bool any = false, all = true;
        for (int d = 0; d < D; ++d) {
            any = any || a.period[d] > 0.0;
            all = all && a.period[d] > 0.0;
        }
        const int per = all ? kPerAll : (any ? kPerMixed : kPerNone);
        if (a.nq <= kQmCompactMax) {
            const dim3 g(b.nchunk, (unsigned)std::min<int64_t>(a.nq, kQmSlots));
            if (per == kPerAll) hipLaunchKernelGGL((k_hill_shared_qm<D, kPerAll, true>), g, dim3(kBlock), 0, s, b);
            else if (per == kPerNone) hipLaunchKernelGGL((k_hill_shared_qm<D, kPerNone, true>), g, dim3(kBlock), 0, s, b);
            else hipLaunchKernelGGL((k_hill_shared_qm<D, kPerMixed, true>), g, dim3(kBlock), 0, s, b);
        } else {
            const dim3 g(b.nchunk, (unsigned)a.nq);
            if (per == kPerAll) hipLaunchKernelGGL((k_hill_shared_qm<D, kPerAll, false>), g, dim3(kBlock), 0, s, b);
            else if (per == kPerNone) hipLaunchKernelGGL((k_hill_shared_qm<D, kPerNone, false>), g, dim3(kBlock), 0, s, b);
            else hipLaunchKernelGGL((k_hill_shared_qm<D, kPerMixed, false>), g, dim3(kBlock), 0, s, b);
        }
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        if (small_finalize(b))
            hipLaunchKernelGGL((k_hill_shared_finalize_wave<D>), dim3((unsigned)a.nq), dim3(64), 0, s, b);
        else
            hipLaunchKernelGGL((k_hill_shared_finalize_wg<D>), dim3((unsigned)a.nq), dim3(kBlock), 0, s, b);
        return hipGetLastError();
    }
    SharedArgs b = a;
    int Q, ql;
    shared_shape(a.nq, a.cap, Q, ql);
    for (b.lg = 0; (ql << b.lg) < 64;) ++b.lg;
    // many chunks: one wavefront (or workgroup) reads a query's records, kept
    // next to each other; few: a lane per query reads them chunk after chunk
    const bool per_query = a.nchunk >= 32;
    b.rec_ch = per_query ? 1 : a.nq;
    b.rec_q = per_query ? a.nchunk : 1;
    const dim3 grid(a.nchunk, (unsigned)((a.nq + ql * Q - 1) / (ql * Q)));
    if (cv && !shared_sums_cvs(a)) return hipErrorInvalidValue;
    switch (Q) {
    case 1: launch_sum<D, 1>(b, cv, grid, s); break;
    case 2: launch_sum<D, 2>(b, cv, grid, s); break;
    case 4: launch_sum<D, 4>(b, cv, grid, s); break;
    default: return hipErrorInvalidValue;
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if (per_query && small_finalize(b))
        hipLaunchKernelGGL((k_hill_shared_finalize_wave<D>), dim3((unsigned)a.nq), dim3(64), 0, s, b);
    else if (per_query)
        hipLaunchKernelGGL((k_hill_shared_finalize_wg<D>), dim3((unsigned)a.nq), dim3(kBlock), 0, s, b);
    else
        hipLaunchKernelGGL((k_hill_shared_finalize<D>), dim3((unsigned)((a.nq + kBlock - 1) / kBlock)), dim3(kBlock),
                           0, s, b);
    return hipGetLastError();
}

}  // namespace

// one chunk per stage of the capacity, and no more than the partial records hold
int64_t most_chunks(int64_t cap, int64_t nq)
{
    return std::min<int64_t>((cap + kStage - 1) / kStage, kMaxRecords / std::max<int64_t>(1, nq));
}

int64_t shared_records(int64_t cap, int64_t nq) { return std::max<int64_t>(1, most_chunks(cap, nq)) * nq; }

// Every workgroup has an equal share of the hills and the queries, so the
// chunks are chosen to give each of the 256 CUs the same number of
// workgroups: k = 4 by default (8 with 4 queries per lane, the longest
// sums), fewer where the capacity has too few stages.  256
// walkers on 100,000 hills, us per step: 27.6 (k = 1), 23.7 (2), 22.6 (3),
// 22.8 (4), 24.3 (6), 25.1 (8); 100 walkers on 50,000 hills in three CVs:
// 14.9 at 2 x 256 workgroups, 16.7 at 548.  8,192 points on 100,000 hills with
// Q = 4: 365.6 (k = 4), 357.6 (8); with Q = 2 369.9 and 363.6, but 28.8 and
// 30.3 for 4,096 points on 10,000.
int32_t shared_chunks(int64_t cap, int64_t nq, int32_t target)
{
    constexpr int kCus = 256;
    int Q, ql;
    shared_shape(nq, cap, Q, ql);
    const int64_t nqb = std::max<int64_t>(1, (nq + (int64_t)ql * Q - 1) / ((int64_t)ql * Q));
    if (target > 0)  // the caller's number, rounded up to whole chunks
        return (int32_t)std::max<int64_t>(1, std::min((cap + kStage - 1) / kStage, (target + nqb - 1) / nqb));
    const int64_t most = most_chunks(cap, nq);
    int64_t nc = most;
    for (int64_t k = Q == 4 ? 8 : 4; k >= 1; --k)
        if (k * kCus / nqb <= most) {
            nc = k * kCus / nqb;
            break;
        }
    return (int32_t)std::max<int64_t>(1, std::min(nc, most));
}

bool shared_sums_cvs(const SharedArgs &a) { return periodic_form(a) == all_periodic(a.D); }

hipError_t launch_hill_shared(const SharedArgs &a, hipStream_t s, const SharedCv *cv)
{
    switch (a.D) {
    case 1: return launch_shared_d<1>(a, cv, s);
    case 2: return launch_shared_d<2>(a, cv, s);
    case 3: return launch_shared_d<3>(a, cv, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace sx
