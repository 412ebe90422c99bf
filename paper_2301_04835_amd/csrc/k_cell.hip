// Coordination numbers with a hard cutoff through cell lists (the switching
// form s(r) = (1 - (r/r0)^n) / (1 - (r/r0)^m), minimum image in an
// orthorhombic periodic box; CVs of this kind extend the paper's CV set,
// Sec. 2.2).  For groups of tens of thousands of atoms the all-pairs
// evaluation gives way to:
//
//   k_cell_build   one workgroup per (walker, group): the cell of every
//                  member (positions wrapped into the box), LDS counts, an
//                  exclusive scan, and a placement in member order within
//                  a cell, so every later sum runs in a fixed order; each
//                  member is stored as (x, y, z) relative to its cell's
//                  origin (float, ~6e-8 nm) and its atom index, and its
//                  sorted position is kept in member order.
//   k_cell_jac     one workgroup per (walker, group, column block of cells
//                  in z): the partner group's members in the cells around
//                  the block are staged in LDS relative to the block's
//                  origin (a cell's offset is its cell step times the cell
//                  edge, periodic wrap included), slice by slice, so each
//                  home cell's neighbours form one contiguous range; a
//                  wavefront takes 16 home atoms against their range: FP32
//                  pair terms, the switch sum (the CV value, on the A side)
//                  and the gradient sum_j f(r_ij)(r_i - r_j) of each (CV,
//                  side) use, stored per member (no atomics, fixed order).
//   k_cn_cell_fin  per (walker, CV): the column-block partials in order.
//   k_cell_gather  the vector-Jacobian product from the stored gradients,
//                  one lane per member in member order (groups identical
//                  or disjoint: one writer per atom).

// Cut-length cells (edge >= the cutoff, >= 3 per dimension) are cut into rz = 4
// sub-cells in z, so the 9 (2 rz + 1) neighbour sub-cells of a sub-cell are
// distinct and hold exactly the one image of every partner within the cutoff.
// The sub-cells shrink the partners a home atom visits from 27 cut-length cubes
// to 9 (2 rz + 1) / rz = 20.3 (6.4 cut spheres' worth of volume to 4.8).
#include <algorithm>

#include "sx_internal.h"
#include "dev_cv.h"
#include "dev_reduce.h"

namespace sx {
namespace {

typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kBuildBlock = 1024;
constexpr int kBuildWords = 20448;  // LDS words of the counting build: the cells', then a 16-bit slot per member
static_assert(kBuildWords >= kCellTotal, "every cell has a word");

// The cell of a coordinate and the position within it (iclen = 1 / clen, its
// rounding made good by the position).
__device__ __forceinline__ int cell_of(double x, double L, double iL, double clen, double iclen, int nc, double &rel)
{
    const double xw = x - L * floor(x * iL);  // into [0, L)
    int c = (int)(xw * iclen);
    c = c < 0 ? 0 : (c >= nc ? nc - 1 : c);
    rel = xw - c * clen;
    const int d = rel < 0.0 && c > 0 ? -1 : (rel >= clen && c < nc - 1 ? 1 : 0);
    if (d != 0) {  // rare
        c += d;
        rel = xw - c * clen;
    }
    return c;
}

// Two ways to place members in member order within their cells.
//
// Turns: of 1,024 members at a time a wavefront finds each lane's cell mates
// among its 64 (bit by bit of the cells' numbers, with ballots) and the 16
// wavefronts go one after the other, each taking its cells' next places: a
// chain of 16 LDS round trips, with the next members' loads and the last ones'
// stores in flight beside it.  (With 64 shuffles a rank and barriers that wait
// for memory too, 20,000 members took 127 us, now 77.)
//
// Counting (SMALL: a 16-bit slot per member fits in LDS next to the cells'
// words, 80 KB, two workgroups a CU): members take the slots of their cell in
// any order (an LDS atomic), then each counts the earlier members among its
// cell's: the place in member order, whatever the slots were.  The records
// requested ahead of the counts are vectors of the language: as float4 they
// waited in scratch memory (96 groups of 20,000 members 71 us, 62 now).
//
// Counting costs a cell the square of its members: the turns serve groups whose
// cells' squares add up to more than crowded() per member (a dense droplet in a
// large box, whose cells are capped at 16 a side).  Counting and turns, us:
//   20,000 members, squares of 4 / 11 / 56 / 186   47 50 95 176   72
//    8,000, squares of 5 / 23 / 32 / 52            24 30 32 44    34
//    5,000, squares of 3 / 15 / 20 / 33            21 25 26 32    26
//    2,000, squares of 2 / 9 / 14 / 20             14 15 17 17    16
// Slots in memory, where they don't fit, were slower than the turns at any
// density (20,000 members in 16,384 cells, squares of 5: 99 and 82).
__device__ __forceinline__ float crowded(int32_t n) { return fminf(35.f, (float)n * (1.f / 256)); }

// A barrier that orders LDS alone: loads and stores of memory stay in flight.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

template <typename T, bool SMALL>
__global__ void __launch_bounds__(kBuildBlock, 8) k_cell_build(CellArgs c, PosView pos)
{
    // a cell's count, first slot, end; then (SMALL) the slots' members
    __shared__ int32_t s_off[SMALL ? kBuildWords : kCellTotal];
    __shared__ int32_t s_tot[kBuildBlock / 64];
    __shared__ float s_sq[kBuildBlock / 64];
    const int w = blockIdx.x / c.G, g = blockIdx.x % c.G;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int32_t n = c.goff[g + 1] - c.goff[g];
    const int32_t *ga = c.gatoms + c.goff[g];
    const int64_t aoff = c.atom_off[w];
    int32_t *cid = c.cid + (int64_t)w * c.gtotal + c.goff[g];
    int32_t *cst = c.cstart + ((int64_t)w * c.G + g) * (c.ncell + 1);
    float4 *srt = c.sorted + (int64_t)w * c.gtotal + c.goff[g];
    float4 *tmp = c.jac + (int64_t)w * c.jtotal + c.joff[g][0];  // records the pair pass writes later
    for (int i = tid; i < c.ncell; i += kBuildBlock) s_off[i] = 0;
    __syncthreads();
    // cells, counts and positions in their cells, four members per thread at a
    // time with their loads issued together (a member past the group's end is
    // member b instead and is dropped)
    for (int32_t b = tid; b < n; b += 4 * kBuildBlock) {
        int32_t a[4];
        double3 r[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int32_t i = b + k * kBuildBlock;
            a[k] = ga[i < n ? i : b];
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) r[k] = ld_pos_t<T>(pos, aoff + a[k]);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int32_t i = b + k * kBuildBlock;
            if (i >= n) break;
            double rx, ry, rz;
            const int cx = cell_of(r[k].x, c.L[0], c.inv_L[0], c.clen[0], c.inv_clen[0], c.nc[0], rx);
            const int cy = cell_of(r[k].y, c.L[1], c.inv_L[1], c.clen[1], c.inv_clen[1], c.nc[1], ry);
            const int cz = cell_of(r[k].z, c.L[2], c.inv_L[2], c.clen[2], c.inv_clen[2], c.nc[2], rz);
            const int cell = (cx * c.nc[1] + cy) * c.nc[2] + cz;
            cid[i] = cell;
            tmp[i] = make_float4((float)rx, (float)ry, (float)rz, __int_as_float(a[k]));
            atomicAdd(&s_off[cell], 1);
        }
    }
    __syncthreads();
    // exclusive scan of the counts: consecutive cells per thread, the threads
    // of a wavefront, the wavefronts in order
    const int per = (c.ncell + kBuildBlock - 1) / kBuildBlock;
    const int c0 = min(tid * per, c.ncell), c1 = min(c0 + per, c.ncell);
    int32_t sum = 0;
    float sq = 0.f;  // the sum of the counts' squares, the same in every thread below
    for (int cc = c0; cc < c1; ++cc) {
        const int32_t m = s_off[cc];
        sum += m;
        sq += (float)m * (float)m;
    }
    int32_t run = sum;
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t y = __shfl_up(run, o, 64);
        if (lane >= o) run += y;
        sq += __shfl_xor(sq, o, 64);
    }
    if (lane == 63) {
        s_tot[wave] = run;
        s_sq[wave] = sq;
    }
    __syncthreads();
    run -= sum;
    sq = 0.f;
    for (int k = 0; k < kBuildBlock / 64; ++k) {
        run += k < wave ? s_tot[k] : 0;
        sq += s_sq[k];
    }
    for (int cc = c0; cc < c1; ++cc) {
        const int32_t m = s_off[cc];
        s_off[cc] = run;
        cst[cc] = run;
        run += m;
    }
    if (tid == 0) cst[c.ncell] = n;
    __syncthreads();
    if (!SMALL || sq > crowded(n) * (float)n) {  // uniform
        // a chunk's cells and records are requested ahead of the turns before it
        int cell = tid < n ? cid[tid] : -1;
        float4 v = tmp[tid < n ? tid : 0];
        for (int32_t base = 0; base < n; base += kBuildBlock) {
            const int32_t i = base + tid, in = i + kBuildBlock;
            const bool valid = i < n;
            const int next_cell = in < n ? cid[in] : -1;
            const float4 next_v = tmp[in < n ? in : 0];
            // the lanes of this lane's cell, bit by bit of its number; how many,
            // and how many of them before it
            uint64_t same = __ballot(valid);
#pragma unroll
            for (int b = 0; (kCellTotal - 1) >> b; ++b) {
                const bool bit = (cell >> b) & 1;
                const uint64_t m = __ballot(bit);
                same &= bit ? m : ~m;
            }
            const int cnt = __popcll(same), rank = __popcll(same & ((1ull << lane) - 1));
            int dst = 0;
            for (int t = 0; t < kBuildBlock / 64; ++t) {
                lds_barrier();
                if (wave == t && valid) {
                    dst = s_off[cell] + rank;
                    if (rank == cnt - 1) s_off[cell] = dst + 1;  // after every lane of the wavefront read it
                }
            }
            if (valid) {
                srt[dst] = v;
                cid[i] = dst;  // from here on: the member's sorted position
            }
            cell = next_cell;
            v = next_v;
        }
        return;
    }
    uint16_t *s_slot = reinterpret_cast<uint16_t *>(s_off + c.ncell);
    for (int32_t b = tid; b < n; b += 4 * kBuildBlock) {
        int32_t cell[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) cell[k] = cid[b + k * kBuildBlock < n ? b + k * kBuildBlock : b];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int32_t i = b + k * kBuildBlock;
            if (i >= n) break;
            s_slot[atomicAdd(&s_off[cell[k]], 1)] = (uint16_t)i;
        }
    }
    __syncthreads();
    // four members' counts side by side, two slots a word: all of the cell's
    // words, less what its first and last hold of the neighbour cells.  A member
    // that is not there (past the group's end) is the thread's first: no other
    // thread's, which may be done with it.
    const uint32_t *s_two = reinterpret_cast<const uint32_t *>(s_slot);
    for (int32_t b = tid; b < n; b += 4 * kBuildBlock) {
        int32_t m[4], lo[4], hi[4], dst[4], len = 0;
        f32x4 v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            m[k] = b + k * kBuildBlock < n ? b + k * kBuildBlock : b;
            lo[k] = cid[m[k]];
            v[k] = *reinterpret_cast<const f32x4 *>(tmp + m[k]);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            hi[k] = s_off[lo[k]];
            dst[k] = lo[k] = lo[k] > 0 ? s_off[lo[k] - 1] : 0;
            len = max(len, ((hi[k] + 1) >> 1) - (lo[k] >> 1));
            dst[k] -= (lo[k] & 1) && s_slot[lo[k] - 1] < m[k] ? 1 : 0;
            dst[k] -= (hi[k] & 1) && s_slot[hi[k]] < m[k] ? 1 : 0;
        }
        for (int32_t q = 0; q < len; ++q)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int32_t e = (lo[k] >> 1) + q, last = (hi[k] - 1) >> 1;
                const uint32_t two = s_two[min(e, last)] | (e > last ? ~0u : 0u);
                dst[k] += ((two & 0xffffu) < (uint32_t)m[k] ? 1 : 0) + ((two >> 16) < (uint32_t)m[k] ? 1 : 0);
            }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            if (b + k * kBuildBlock < n) {
                *reinterpret_cast<f32x4 *>(srt + dst[k]) = v[k];
                cid[m[k]] = dst[k];  // from here on: the member's sorted position
            }
        }
    }
}

// Is the pair within the cut?  Far from its edge the FP32 distance decides.
// Within 1e-5 of it the pair is decided from the positions as given, in
// FP64, one operation at a time and without contraction: d = a - b,
// d -= L rint(d / L), r = sqrt((dx^2 + dy^2) + dz^2), inside unless r >= rcut
// (the plain definition of the minimum-image cut, so that a pair at the
// edge falls on the same side as under that definition).  Out of line: the
// path is rare and keeps its registers out of the pair loop.
__device__ __attribute__((noinline)) bool cut_exact(PosView pos, int64_t aoff, int32_t ai, int32_t aj, double L0,
                                                   double L1, double L2, double rcut)
{
#pragma clang fp contract(off)
    const double3 p = ld_pos(pos, aoff + ai), q = ld_pos(pos, aoff + aj);
    double dx = p.x - q.x, dy = p.y - q.y, dz = p.z - q.z;
    dx = dx - L0 * rint(dx / L0);
    dy = dy - L1 * rint(dy / L1);
    dz = dz - L2 * rint(dz / L2);
    const double r = sqrt(dx * dx + dy * dy + dz * dz);
    return !(r >= rcut);
}

__device__ __forceinline__ const CvDesc &cell_cv(const CvSet &cs, int k)
{
    int c = 0;
    for (; c < cs.ncv - 1; ++c)
        if (cs.cv[c].kind == CV_COORD_CELL && cs.cv[c].cn == k) break;
    return cs.cv[c];
}

// Stage the members of group gp in the region of column block (cx, cy, z0):
// the 3 x 3 x (czb + 2 rz) sub-cells around it, slice by slice (z offset -rz
// .. czb + rz - 1), each slice in (x, y) order, so that the neighbour
// sub-cells of the block's k-th home sub-cell (z offsets -rz .. rz around it)
// are the contiguous range s_seg[9 k] .. s_seg[9 (k + 2 rz + 1)].  Positions
// relative to the origin of cell (cx, cy, z0), times sc, and their squared
// length; entries [r0, r0 + kColStage) of the region, behind kFar entries and
// followed by kTiles tiles outside any cut.  Returns how many are real.  Its
// loads are waited for, not its instructions: with a sub-cell's two starts and
// eight of its members in flight per thread instead of one load at a time the
// pair pass without its pairs took 483 us, 514 before.
constexpr int kJacBlock = 256;
constexpr int kTile = 16;                       // home atoms of a wavefront, partners of a tile
constexpr int kApp = kTile * kJacBlock / 64;    // home atoms per pass
constexpr int kColStage = 1728;                 // partner atoms staged per round (28 KB: five workgroups a CU)
constexpr int kTiles = 8;                       // tiles tested per step: one 32-bit mask
constexpr int kFar = 4;                         // partners beyond every cut ahead of the staged ones
constexpr int kStageLd = kFar + kColStage + kTiles * kTile + 12;  // with a step of padding
static_assert(kStageLd % 64 == 16, "the four coordinates' reads of a tile hit different banks");
constexpr int kLoads = 8;                       // members of a sub-cell in flight per thread
constexpr int kSide = 3, kXY = kSide * kSide;  // neighbour cells in x (y), in a layer
constexpr int kRegMax = kXY * (kCzMax + 2 * kZReach);
constexpr int kRegPer = (kRegMax + kJacBlock - 1) / kJacBlock;  // region sub-cells per thread

// i + o wrapped into [0, n) for -n <= i + o < 2n (no division)
__device__ __forceinline__ int wrap_cell(int v, int n)
{
    v += v < 0 ? n : 0;
    return v >= n ? v - n : v;
}

struct Staged {
    float c[4][kStageLd];  // x, y, z, x^2 + y^2 + z^2
};

__device__ __forceinline__ int stage_column(const CellArgs &c, int w, int gp, int cx, int cy, int z0, int czb, int r0,
                                            float sc, float lim, Staged &sp, int32_t *s_seg,
                                            int32_t *s_first, int32_t *s_wsum, int32_t *s_odd)
{
    const int32_t *cst = c.cstart + ((int64_t)w * c.G + gp) * (c.ncell + 1);
    const float4 *srt = c.sorted + (int64_t)w * c.gtotal + c.goff[gp];
    const int nreg = kXY * (czb + 2 * c.rz);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) *s_odd = 0;
    // thread tid's sub-cells are tid, tid + 256, ..: first sorted member and
    // member count, all loads in flight together; then an exclusive scan of
    // the counts, inside each wavefront and over the wavefronts' totals in order
    constexpr int kWaves = kJacBlock / 64;
    int n[kRegPer], x[kRegPer];
#pragma unroll
    for (int q = 0; q < kRegPer; ++q) {
        const int t = q * kJacBlock + tid;
        n[q] = 0;
        if (t < nreg) {
            const int sl = t / kXY, xy = t % kXY;
            const int ox = xy / kSide - 1, oy = xy % kSide - 1, oz = sl - c.rz;
            // |ox|, |oy| <= 1 < nc and -rz <= z0 + oz < nc2 + rz with rz <= nc2
            const int nx = wrap_cell(cx + ox, c.nc[0]), ny = wrap_cell(cy + oy, c.nc[1]);
            const int nz = wrap_cell(z0 + oz, c.nc[2]);
            const int nb = (nx * c.nc[1] + ny) * c.nc[2] + nz;
            const int f = cst[nb];
            n[q] = cst[nb + 1] - f;
            s_first[t] = f;
        }
    }
#pragma unroll
    for (int q = 0; q < kRegPer; ++q) {
        if (q * kJacBlock >= nreg) break;  // uniform
        x[q] = n[q];
        for (int o = 1; o < 64; o <<= 1) {
            const int y = __shfl_up(x[q], o, 64);
            if (lane >= o) x[q] += y;
        }
        if (lane == 63) s_wsum[q * kWaves + wave] = x[q];
    }
    __syncthreads();
    int total = 0;
#pragma unroll
    for (int q = 0; q < kRegPer; ++q) {
        if (q * kJacBlock >= nreg) break;
        int base = total + x[q] - n[q];
#pragma unroll
        for (int wv = 0; wv < kWaves; ++wv) {
            const int ws = s_wsum[q * kWaves + wv];
            base += wv < wave ? ws : 0;
            total += ws;
        }
        const int t = q * kJacBlock + tid;
        if (t < nreg) s_seg[t] = base;
    }
    if (tid == 0) s_seg[nreg] = total;
    __syncthreads();
    // the window [r0, r0 + m) of the region, sub-cell by sub-cell: each
    // member shifted by its sub-cell's offset from the block origin
    const int m = min(kColStage, total - r0);
    for (int t = tid; t < nreg; t += blockDim.x) {
        const int sg = s_seg[t];
        const int e0 = max(sg, r0), e1 = min(s_seg[t + 1], r0 + m);
        if (e0 >= e1) continue;
        const int f = s_first[t];
        const int sl = t / kXY, xy = t % kXY;
        const int ox = xy / kSide - 1, oy = xy % kSide - 1, oz = sl - c.rz;
        const float shx = (float)(ox * c.clen[0]), shy = (float)(oy * c.clen[1]), shz = (float)(oz * c.clen[2]);
        for (int eb = e0; eb < e1; eb += kLoads) {  // past the last member: its copy, dropped
            float4 v[kLoads];
#pragma unroll
            for (int l = 0; l < kLoads; ++l) v[l] = srt[f + (min(eb + l, e1 - 1) - sg)];
#pragma unroll
            for (int l = 0; l < kLoads; ++l) {
                const int e = eb + l;
                if (e >= e1) break;
                const float px = (v[l].x + shx) * sc, py = (v[l].y + shy) * sc, pz = (v[l].z + shz) * sc;
                sp.c[0][kFar + e - r0] = px;
                sp.c[1][kFar + e - r0] = py;
                sp.c[2][kFar + e - r0] = pz;
                const float p2 = fmaf(px, px, fmaf(py, py, pz * pz));
                sp.c[3][kFar + e - r0] = p2;
                if (!(p2 <= lim)) *s_odd = 1;  // not a position of the region (NaN): no cull in this window
            }
        }
    }
    if (tid < kFar + kTiles * kTile) {
        const int e = tid < kFar ? tid : m + tid;
        sp.c[0][e] = sp.c[1][e] = sp.c[2][e] = 1e9f;
        sp.c[3][e] = 1e30f;
    }
    __syncthreads();
    return m;
}

// One workgroup of 256 threads per (column block, group, walker).  A
// wavefront takes 16 home atoms at a time (the members of the block's cells,
// contiguous in the sorted order) and, for every use (CV, partner group) of
// the group, the union of their home cells' contiguous partner ranges (what it
// adds to an atom's own range lies beyond the cut) in two passes:
//
//   cull  four in five candidates lie outside the cut.  A tile of 16 partners
//         against the 16 home atoms is one v_mfma_f32_16x16x4_f32,
//         D = |p|^2 - 2 p.o + (|o|^2 - R^2), R^2 the squared cut plus the
//         product's rounding error (below 8 2^-24 (|o| + |p|)^2), so no pair
//         that the float32 or the exact decision counts is lost; a window with
//         a position outside that bound (no number) keeps every pair.  A lane
//         holds home atom lane % 16 and four partners of the tile; the signs
//         of eight tiles are its 32-bit word;
//   pairs the kept partners, two at a time: FP32 differences, the switch sum
//         (A side of the CV: the CV value) and the gradient sum
//         sum_j f(r_ij) (r_i - r_j).
//
// The atom's four lanes combine in a fixed butterfly and the gradient is
// stored per member and use (the VJP reads it).  A group's own CV counts its
// self pair (r = 0: s = 1 exactly, zero gradient), so the A-side sum drops 1
// per atom instead of testing every pair.
//
// With every candidate evaluated in FP32 (19 operations and a 16-byte LDS read
// each, 8 lanes an atom) the pass was bound by VALU issue and LDS reads: 32
// walkers of 60,000 atoms in three groups and three CVs took 1,287 us; with a
// cull on the vector units (7 operations, three LDS words) 982, with this one
// (one LDS word per lane and four shifts for 256 tests) 926, with the lanes'
// words queued one deep so that a wavefront waits for its fullest lane over
// the range and not per word 897, and with far partners in place of masked
// lanes (52 instructions for two pairs, 66 before) 868.  VALU issue still
// bounds it: 1 in 3 instructions belongs to the cull, and of the pair
// loop's lanes 2 in 3 hold a pair.
struct PairCtx {
    float rc2s, bandcs, rc2;  // squared cut and its band in the units of t, squared cut
    float cull2;              // R^2
    int64_t aoff;
    const float4 *srt;        // the partner group's sorted members
    const int32_t *s_seg, *s_first;
    int nreg, r0;             // region sub-cells, first entry of the staged window
    float lim;                // largest |o|^2, |p|^2 that the cull's error bound covers
};

// The atom index of staged entry e of the region (rare: the exact cut
// decision): its sub-cell by bisection of the region's starts.
__device__ __attribute__((noinline)) int32_t staged_atom(const float4 *srt, const int32_t *s_seg,
                                                        const int32_t *s_first, int nreg, int e)
{
    int lo = 0, hi = nreg - 1;  // the last sub-cell that starts at or before e
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (s_seg[mid] <= e) lo = mid; else hi = mid - 1;
    }
    return __float_as_int(srt[s_first[lo] + (e - s_seg[lo])].w);
}

// Two kept partners of one home atom (o), at byte offsets e of the staged
// arrays (a far partner in the place of a missing one: it adds zero).  The
// cut decision, the switch sum and the gradient sum.  In the (6, 12) form the
// coordinates are in units of r0 (x^2 = r^2 / r0^2 directly) and the gradient
// term is x^4 s^2 (r_i - r_j) / r0, the factor -6 / r0 applied once per atom;
// otherwise plain units and f of switch_fn.  SIDEA: the switch sum is wanted
// (the A side of the CV); on the B side only the gradient is.
//
// The cut enters the (6, 12) switch without a select: t = (r^2 - rc^2) 2^100
// (one fma; scaling by a power of two keeps the rounding of r^2 - rc^2, so
// the decision and its band are those of the unscaled difference), and
// s = 1 / max(1 + x^6, t).  Inside the cut t < 0 and s is the switch; a
// partner decided outside (outside the band) has t > 2^100 * 1e-5 rc^2
// (rc^2 in r0 units: 7e25 at rc = 2.4 r0, above 3e24 for any cut beyond
// r0 / 2), so s < 3e-25 and x^4 s^2 underflows to zero or a denormal: it
// adds nothing measurable to the gradient and less than 3e-25 to the switch
// sum, far below the sum's last bit.  A partner that the exact decision
// drops gets t = +inf, s = 0; a far one (1e9) has t = +inf by itself.
constexpr float kTScale = 0x1p100f;

struct HomeSum {  // of one home atom
    float s, x, y, z;
};

// coordinate d of the staged entry at byte offset e
__device__ __forceinline__ float staged(const Staged &sp, int d, int e)
{
    return *reinterpret_cast<const float *>(reinterpret_cast<const char *>(sp.c[d]) + e);
}

template <bool S612, bool SIDEA>
__device__ __forceinline__ void pair2(const Staged &sp, const int (&e)[2], float3 o, int32_t me,
                                      const PairCtx &k, const CvDesc &cv, const CellArgs &c, const PosView &pos,
                                      HomeSum &g)
{
    float dx[2], dy[2], dz[2], r2[2], t[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        dx[q] = o.x - staged(sp, 0, e[q]);
        dy[q] = o.y - staged(sp, 1, e[q]);
        dz[q] = o.z - staged(sp, 2, e[q]);
        r2[q] = fmaf(dx[q], dx[q], fmaf(dy[q], dy[q], dz[q] * dz[q]));
        t[q] = S612 ? fmaf(r2[q], kTScale, -k.rc2s) : r2[q] - k.rc2;
    }
    if (fminf(fabsf(t[0]), fabsf(t[1])) <= k.bandcs) {  // rare: the edge of the cut
#pragma unroll
        for (int q = 0; q < 2; ++q)
            if (fabsf(t[q]) <= k.bandcs)
                t[q] = cut_exact(pos, k.aoff, me, staged_atom(k.srt, k.s_seg, k.s_first, k.nreg, k.r0 + e[q] / 4 - kFar), c.L[0],
                                 c.L[1], c.L[2], cv.rcut)
                           ? -1.0f
                           : __builtin_inff();
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        float f;
        if (S612) {
            const float x4 = r2[q] * r2[q];
            // max(1 + x^6, t) on the bit patterns: 1 + x^6 is positive, so
            // the signed-integer order agrees with the float order here
            const float den = __int_as_float(max(__float_as_int(fmaf(x4, r2[q], 1.0f)), __float_as_int(t[q])));
            const float sv = __builtin_amdgcn_rcpf(den);
            if (SIDEA) g.s += sv;
            f = x4 * sv * sv;
        } else {
            const bool in = t[q] < 0.f;
            float sv;
            switch_fn(r2[q], cv, sv, f);
            if (SIDEA) g.s += in ? sv : 0.f;
            f = in ? f : 0.f;
        }
        g.x = fmaf(f, dx[q], g.x);
        g.y = fmaf(f, dy[q], g.y);
        g.z = fmaf(f, dz[q], g.z);
    }
}

// Partners [b0, b1) of the staged window (uniform per wavefront) against its
// 16 home atoms; live: this lane's atom counts.  bo: the lane's word of the
// home operand, (-2 x, -2 y, -2 z, 1) by lane / 16; co = |o|^2 - R^2.
// odd: no cull (a position in the window or o is outside its bound).
template <bool S612, bool SIDEA>
__device__ __forceinline__ void home_pairs(const Staged &sp, int b0, int b1, float3 o, float bo, float co, bool live,
                                           bool odd, int32_t me, const PairCtx &k, const CvDesc &cv,
                                           const CellArgs &c, const PosView &pos, HomeSum &g)
{
    const int lane = threadIdx.x & 63, quad = lane >> 4;
    // row r of a tile is its partner 4 (r % 4) + r / 4, so that a lane's rows
    // 4 quad + v are the partners quad + 4 v: an atom's lanes take every
    // fourth partner and keep about as many each
    const float *const pa = &sp.c[quad][kFar + 4 * (lane & 3) + ((lane & 15) >> 2)];
    const f32x4 cc = {co, co, co, co};
    if (b0 >= b1) return;  // none of the atoms' ranges in this window (uniform): b0 may lie past its end
    uint32_t m0 = 0, m1 = 0;  // kept partners of the lane's current word and of the next
    int e0 = 0;               // byte offset of bit 0 of m0 in a staged array
    float a[kTiles];
#pragma unroll
    for (int t = 0; t < kTiles; ++t) a[t] = pa[b0 + t * kTile];
    for (int j = b0; j < b1; j += kTiles * kTile) {
        // eight tiles; a tile at or past b1 holds partners beyond every cut,
        // or padding
        f32x4 D[kTiles];
#pragma unroll
        for (int t = 0; t < kTiles; ++t) D[t] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[t], bo, cc, 0, 0, 0);
        const int jn = j + kTiles * kTile;
        if (jn < b1) {  // uniform: the next tiles' words, in flight during this mask's pairs
#pragma unroll
            for (int t = 0; t < kTiles; ++t) a[t] = pa[jn + t * kTile];
        }
        uint32_t m = 0;  // bit i: partner quad + 4 i of the word's
#pragma unroll
        for (int t = kTiles - 1; t >= 0; --t)
#pragma unroll
            for (int v = 3; v >= 0; --v)
                m = __builtin_amdgcn_alignbit(m, __float_as_uint(D[t][v]), 31);  // 2 m + (D < 0)
        if (odd) {  // all of [j, b1)
            const int n = (b1 - j - quad + 3) >> 2;
            m = n <= 0 ? 0u : (n >= 32 ? ~0u : (1u << n) - 1u);
        }
        // the word waits behind the lane's last one, so that lanes with few
        // partners in one word run ahead into the next; after the last word
        // both drain.  A lane without a partner takes a far one.
        m1 = live ? m : 0u;
        const bool last = jn >= b1;
        for (;;) {
            const bool next = m0 == 0;
            m0 = next ? m1 : m0;
            m1 = next ? 0u : m1;
            e0 = next ? 4 * (kFar + j + quad) : e0;
            if (!__any(last ? m0 != 0 : m1 != 0)) break;  // m1 is empty if m0 is
            int e[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                e[q] = m0 != 0 ? e0 + 16 * __builtin_ctz(m0) : 0;
                m0 &= m0 - 1u;
            }
            pair2<S612, SIDEA>(sp, e, o, me, k, cv, c, pos, g);
        }
    }
}

template <bool S612>
__global__ void __launch_bounds__(kJacBlock, 5) k_cell_jac(CellArgs c, CvSet cs, PosView pos)
{
    __shared__ Staged s_p;
    __shared__ int32_t s_seg[kRegMax + 1], s_first[kRegMax], s_wsum[kRegPer * kJacBlock / 64];
    __shared__ double s_red[kJacBlock / 64];
    __shared__ int32_t s_odd;
    __shared__ int32_t s_home[kCzMax + 1];  // sorted position of the block's home cells
    const int blk = blockIdx.x, g = blockIdx.y, w = blockIdx.z;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int zb = blk % c.nzb, cy = (blk / c.nzb) % c.nc[1], cx = blk / (c.nzb * c.nc[1]);
    // blocks split the column evenly: nzb blocks of at most kCzMax cells
    const int z0 = zb * c.nc[2] / c.nzb, czb = (zb + 1) * c.nc[2] / c.nzb - z0;
    const int32_t *cst = c.cstart + ((int64_t)w * c.G + g) * (c.ncell + 1);
    const float4 *sg = c.sorted + (int64_t)w * c.gtotal + c.goff[g];
    const int cell0 = (cx * c.nc[1] + cy) * c.nc[2] + z0;
    if (tid <= czb) s_home[tid] = cst[cell0 + tid];
    __syncthreads();
    const int a0 = s_home[0], a1 = s_home[czb];
    const int64_t aoff = c.atom_off[w];
    const int nreg = kXY * (czb + 2 * c.rz), span = kXY * (2 * c.rz + 1);
    for (int u = 0; u < c.ninv[g]; ++u) {
        const CvDesc &cv = cs.cv[c.inv_cv[g][u]];
        const bool sideA = c.inv_side[g][u] == 0;
        const float self1 = cv.ga == cv.gb ? 1.0f : 0.0f;
        float4 *J = c.jac + (int64_t)w * c.jtotal + c.joff[g][u];
        // coordinate scale, squared cut, its band, and the gradient factor
        const float sc = S612 ? cv.inv_r0 : 1.0f;
        const float rc2 = cv.rcut2 * sc * sc, bandc = 1e-5f * rc2, gsc = S612 ? -6.0f * cv.inv_r0 : 1.0f;
        // the cut test's difference and band in the units of pair2's t
        const float rc2s = S612 ? rc2 * kTScale : rc2, bandcs = S612 ? bandc * kTScale : bandc;
        const float ext = c.ext * sc;  // |o|, |p| <= sqrt(3) ext; the factor below is 8 2^-24 x 12, rounded up
        PairCtx pc{rc2s, bandcs, rc2, rc2 * 1.0001f + 6e-6f * ext * ext, aoff,
                   c.sorted + (int64_t)w * c.gtotal + c.goff[c.inv_p[g][u]], s_seg, s_first, nreg, 0,
                   3.003f * ext * ext};
        double ssum = 0.0;  // this lane's switch sums (A side), over its home atoms
        for (int r0 = 0;; r0 += kColStage) {
            const int m = stage_column(c, w, c.inv_p[g][u], cx, cy, z0, czb, r0, sc, pc.lim,
                                            s_p, s_seg, s_first, s_wsum, &s_odd);
            pc.r0 = r0;
            for (int h0 = a0 + kTile * wave; h0 < a1; h0 += kApp) {  // uniform per wavefront
                const int i = h0 + (lane & 15);
                const bool live = i < a1;
                const float4 pi = sg[live ? i : a1 - 1];  // past the last atom: its copy, dropped
                int kc = 0;  // this atom's home cell within the block: the last kc with s_home[kc] <= i
                for (int hi = czb - 1; kc < hi;) {
                    const int mid = (kc + hi + 1) >> 1;
                    if (s_home[mid] <= min(i, a1 - 1)) kc = mid; else hi = mid - 1;
                }
                // partners in the staged window of the first atom's cell to the last's
                const int kf = __builtin_amdgcn_readlane(kc, 0), kl = __builtin_amdgcn_readlane(kc, 15);
                const int b0 = max(0, s_seg[kXY * kf] - r0), b1 = min(m, s_seg[kXY * kl + span] - r0);
                // home atoms are stored relative to their own cell: the kc-th
                // cell of the block sits kc cell edges above the block origin
                const float3 o = make_float3(pi.x * sc, pi.y * sc, (pi.z + (float)(kc * c.clen[2])) * sc);
                const int quad = lane >> 4;
                const float bo = quad == 3 ? 1.0f : -2.0f * (quad == 0 ? o.x : quad == 1 ? o.y : o.z);
                const float o2 = fmaf(o.x, o.x, fmaf(o.y, o.y, o.z * o.z)), co = o2 - pc.cull2;
                const bool odd = s_odd != 0 || !(o2 <= pc.lim);
                const int32_t me = __float_as_int(pi.w);
                HomeSum gs{0.f, 0.f, 0.f, 0.f};
                if (sideA)
                    home_pairs<S612, true>(s_p, b0, b1, o, bo, co, live, odd, me, pc, cv, c, pos, gs);
                else
                    home_pairs<S612, false>(s_p, b0, b1, o, bo, co, live, odd, me, pc, cv, c, pos, gs);
#pragma unroll
                for (int q = 16; q < 64; q <<= 1) {
                    gs.s += __shfl_xor(gs.s, q, 64);
                    gs.x += __shfl_xor(gs.x, q, 64);
                    gs.y += __shfl_xor(gs.y, q, 64);
                    gs.z += __shfl_xor(gs.z, q, 64);
                }
                if (quad == 0 && live) {
                    float4 gv = make_float4(gs.x * gsc, gs.y * gsc, gs.z * gsc, 0.f);
                    if (r0 > 0) {  // later windows add to the earlier ones (same thread)
                        const float4 pv = J[i];
                        gv.x += pv.x;
                        gv.y += pv.y;
                        gv.z += pv.z;
                    }
                    J[i] = gv;
                    if (sideA) ssum += (double)gs.s - (r0 == 0 ? (double)self1 : 0.0);
                }
            }
            const bool last = r0 + m >= s_seg[nreg];  // uniform
            __syncthreads();  // the next window or use restages
            if (last) break;
        }
        if (sideA) {  // the CV's partial over this block: fixed butterfly, then waves in order
            ssum = wave_sum(ssum);
            if ((tid & 63) == 0) s_red[wave] = ssum;
            __syncthreads();
            if (tid == 0) {
                double t = s_red[0];
                for (int q = 1; q < kJacBlock / 64; ++q) t += s_red[q];
                c.part[((int64_t)w * c.ncn + cv.cn) * c.nblk + blk] = t;
            }
        }
    }
}

// per (walker, CV): the column-block partials of its A side in block order
__global__ void __launch_bounds__(kBlock) k_cn_cell_fin(CellArgs c, CvSet cs, double *xi)
{
    __shared__ double s_red[kBlock / 64];
    const int k = blockIdx.x, w = blockIdx.y;
    const CvDesc cv = cell_cv(cs, k);
    const double *p = c.part + ((int64_t)w * c.ncn + k) * c.nblk;
    double v = 0.0;
    for (int i = threadIdx.x; i < c.nblk; i += kBlock) v += p[i];
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) s_red[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = s_red[0];
        for (int q = 1; q < kBlock / 64; ++q) t += s_red[q];
        xi[(int64_t)w * cs.D + cv.d] = t * (double)cv.scale;
    }
}

// VJP from the stored gradients: one lane per member of each group in
// member order, out += sign sum over the group's uses of coef[cv] scale_cv J,
// J read at the member's sorted position (left in cid by the build); the
// groups are identical or disjoint, so every atom has one writer.  Members
// listed in atom order make the force updates contiguous; the gradient
// reads land anywhere in the walker's records, so all blocks of one walker
// run on one XCD (blocks are dealt to the 8 XCDs in turn): block b serves
// walker 8 (k / nch) + b % 8, chunk k % nch, k = b / 8, and those records
// pass through one L2.
__global__ void __launch_bounds__(kBlock) k_cell_gather(CellArgs c, CvSet cs, const double *coef, double sign,
                                                         ForceView F, int32_t nch)
{
    const int k = blockIdx.x / 8;
    const int w = (k / nch) * 8 + (int)(blockIdx.x % 8);
    const int64_t e = (int64_t)(k % nch) * blockDim.x + threadIdx.x;
    if (w >= c.W || e >= c.gtotal) return;
    int g = 0;
    while (g + 1 < c.G && e >= c.goff[g + 1]) ++g;
    const int32_t atom = c.gatoms[e];
    const int32_t sp = c.cid[(int64_t)w * c.gtotal + e];
    double fx = 0.0, fy = 0.0, fz = 0.0;
    for (int u = 0; u < c.ninv[g]; ++u) {
        const CvDesc &cv = cs.cv[c.inv_cv[g][u]];
        const double cf = sign * coef[(int64_t)w * cs.D + cv.d] * (double)cv.scale;
        const float4 j = c.jac[(int64_t)w * c.jtotal + c.joff[g][u] + sp];
        fx += cf * (double)j.x;
        fy += cf * (double)j.y;
        fz += cf * (double)j.z;
    }
    float *f = F.ptr + (c.atom_off[w] + atom) * F.sa;
    f[0] += (float)fx;
    f[F.sk] += (float)fy;
    f[2 * F.sk] += (float)fz;
}

}  // namespace

hipError_t launch_cell_cv(const CellArgs &c, const CvSet &cs, const PosView &pos, double *xi, hipStream_t s, int which)
{
    if (c.ncn == 0) return hipSuccess;
    hipError_t e = hipSuccess;
    if (which & 1) {
        int32_t nmax = 0;
        for (int g = 0; g < c.G; ++g) nmax = std::max(nmax, c.goff[g + 1] - c.goff[g]);
        // every member's 16-bit number behind the cells' words
        const bool small = nmax <= 65536 && (int64_t)c.ncell + (nmax + 1) / 2 <= kBuildWords;
        const dim3 grid(c.W * c.G), block(kBuildBlock);
        if (pos.f64 && small)
            hipLaunchKernelGGL((k_cell_build<double, true>), grid, block, 0, s, c, pos);
        else if (pos.f64)
            hipLaunchKernelGGL((k_cell_build<double, false>), grid, block, 0, s, c, pos);
        else if (small)
            hipLaunchKernelGGL((k_cell_build<float, true>), grid, block, 0, s, c, pos);
        else
            hipLaunchKernelGGL((k_cell_build<float, false>), grid, block, 0, s, c, pos);
        e = hipGetLastError();
        if (e != hipSuccess || !(which & 2)) return e;
    }
    bool all612 = true;
    for (int d = 0; d < cs.ncv; ++d)
        if (cs.cv[d].kind == CV_COORD_CELL) all612 = all612 && cs.cv[d].n == 6 && cs.cv[d].m == 12;
    const dim3 grid(c.nblk, c.G, c.W);
    if (all612)
        hipLaunchKernelGGL(k_cell_jac<true>, grid, dim3(kJacBlock), 0, s, c, cs, pos);
    else
        hipLaunchKernelGGL(k_cell_jac<false>, grid, dim3(kJacBlock), 0, s, c, cs, pos);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_cn_cell_fin, dim3(c.ncn, c.W), dim3(kBlock), 0, s, c, cs, xi);
    return hipGetLastError();
}

hipError_t launch_cell_vjp(const CellArgs &c, const CvSet &cs, const PosView &, const double *coef, double sign,
                           ForceView out, hipStream_t s)
{
    if (c.ncn == 0) return hipSuccess;
    const int32_t nch = (int32_t)((c.gtotal + kBlock - 1) / kBlock);
    const int64_t nb = (int64_t)nch * ((c.W + 7) / 8) * 8;
    if (nb > INT32_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_cell_gather, dim3((unsigned)nb), dim3(kBlock), 0, s, c, cs, coef, sign, out, nch);
    return hipGetLastError();
}

}  // namespace sx
