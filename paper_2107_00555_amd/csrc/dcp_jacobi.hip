// dcp_jacobi.hip -- the two Jacobi stencil programs the paper lists
// (jacobi_1d, Sec. 2.2; jacobi_2d, Sec. 4.3) on gfx950, and their C ABI.
//
// Each pass of the listings' time loop writes B's interior from A, then A's
// interior from B; the ends (1D) or the outer rows and columns (2D) of both
// arrays are never written.  Every new value is the listing's sum, added left
// to right, times the listing's weight, each operation rounded once (the
// library is built without FP contraction), so the results equal the plain
// serial evaluation bit for bit.
//
// Temporal blocking in registers.  A launch ("pass") applies several
// half-steps to a tile of the arrays plus a halo as wide as the number of
// half-steps, so only the tile's values need to be exact at the end and the
// halo is recomputed redundantly.  The tile's state lives in VGPRs for the
// whole pass: each lane holds a short run of points of both arrays; in-wave
// neighbours come from lane shuffles and (2D) the rows on the edge of a
// wave's band are exchanged through LDS with one barrier per half-step.
// A pass reads A (and B where it is fixed) once and writes both once, so
// the HBM traffic per half-step falls by the number of half-steps per pass.
// Passes read one pair of arrays and write the other (the caller's arrays
// and a workspace copy, in turn); the pass count is even, so the result
// ends in the caller's arrays.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <type_traits>

#include "dcp.h"
#include "dcp_internal.h"

namespace {

constexpr double kW1 = 0.33333;  // jacobi_1d weight, as the listing writes it
constexpr double kW2 = 0.2;      // jacobi_2d weight

// bfix: where B's boundary cells are read (they never change).  write_b:
// 0 = B is not stored (no later pass reads B's interior), 1 = the tile of B
// is stored, 2 = only B's interior cells of the tile are stored (bout is the
// array bfix points to).
struct J1Args {
    const double *ain, *bin, *bfix;
    double *aout, *bout;
    int64_t n, inner;
    int hh, nhalf, phase;  // halo of a region, half-steps in this pass, 1 = first half-step writes A
    int write_b;
    int align;  // regions are placed so that the array's ends start or end a lane's run
};

// vec16: every lane's two columns are one aligned 16-byte pair (n1 and hh
// even, arrays 16-byte aligned), so loads and stores move both at once.
struct J2Args {
    const double *ain, *bin, *bfix;
    double *aout, *bout;
    int64_t n0, n1;
    int inner_r, inner_c, tiles_r;
    int hh, nhalf, phase, write_b, vec16;
};

__device__ __forceinline__ int j_xcd_remap(int b, int nb) {
    // consecutive workgroups go to different XCDs; number the tiles so that
    // an XCD works on a contiguous run of them (neighbouring halos share L2)
    const int per = nb >> 3, rem = nb & 7;
    const int xcd = b & 7, j = b >> 3;
    return xcd * per + min(xcd, rem) + j;
}

// Cross-lane moves within a wave as DPP wavefront shifts (full-rate VALU,
// no LDS round trip).  from_lower: lane i receives x of lane i-1 (lane 0
// receives 0); from_upper: lane i receives x of lane i+1 (lane 63: 0).
template <int CTRL>
__device__ __forceinline__ double j_dpp(double x) {
    const unsigned long long b = __builtin_bit_cast(unsigned long long, x);
    const int lo = __builtin_amdgcn_mov_dpp((int)(unsigned)b, CTRL, 0xF, 0xF, true);
    const int hi = __builtin_amdgcn_mov_dpp((int)(unsigned)(b >> 32), CTRL, 0xF, 0xF, true);
    return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double from_lower(double x) { return j_dpp<0x138>(x); }  // wave_shr:1
__device__ __forceinline__ double from_upper(double x) { return j_dpp<0x130>(x); }  // wave_shl:1

// keep[lane] ? old : nv, as two v_cndmask_b32 (a plain ?: here is turned
// into a branch per cell, which serialises the unrolled update)
__device__ __forceinline__ double j_keep(uint64_t keep, double nv, double old) {
    const uint64_t nb = __builtin_bit_cast(uint64_t, nv), ob = __builtin_bit_cast(uint64_t, old);
    unsigned lo, hi;
    asm("v_cndmask_b32_e64 %0, %1, %2, %3" : "=v"(lo) : "v"((unsigned)nb), "v"((unsigned)ob), "s"(keep));
    asm("v_cndmask_b32_e64 %0, %1, %2, %3"
        : "=v"(hi)
        : "v"((unsigned)(nb >> 32)), "v"((unsigned)(ob >> 32)), "s"(keep));
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}

// Which cells a half-step may overwrite.  Only the array's own boundary
// cells must keep their values: a cell on the region's edge, or outside the
// array, feeds no cell whose value is still needed once it has been
// recomputed from incomplete neighbours (the exact part of the region
// shrinks by one cell per half-step, and the halo is as wide as the pass),
// and the weights sum to at most 1, so such values stay finite.  A region
// with no boundary cell therefore updates every cell with no mask at all.

// ---------------------------------------------------------------- jacobi_1d
// One wave per workgroup; lane l holds the K consecutive points starting at
// region offset l*K.  The region is 64*K points, the first hh and last hh of
// which are the halo; the rest (inner) is this workgroup's tile.  Loads and
// stores go through LDS so that every global access instruction covers 64
// consecutive elements (the run layout is transposed in LDS, with one pad
// element per run so the lanes' runs fall in different banks).
template <int K>
__global__ void __launch_bounds__(64) j1_kernel(J1Args a) {
    constexpr int R = 64 * K;
    __shared__ double stage[64 * (K + 1)];
    const int lane = threadIdx.x;
    const int64_t n = a.n;
    // Global index of region cell 0.  With a.align (arrays whose waves all run
    // at once, so that a pass is as long as its slowest wave) a region that holds
    // the array's last cell moves left until that cell ends a lane's run; the
    // first cell starts one (a.hh and a.inner are whole runs then, and a.hh has
    // room for the move).
    int64_t rbase = (int64_t)blockIdx.x * a.inner - a.hh;
    const int64_t own0 = rbase + a.hh;  // the tile: [own0, own0 + inner)
    if (a.align && rbase + R >= n) {
        const int64_t m = (rbase - n) % K;
        rbase -= m < 0 ? m + K : m;
    }
    const int64_t g0 = rbase + (int64_t)lane * K;
    auto pos = [](int i) { return i + i / K; };

    // cells outside the array read its nearest end: they only feed the end
    // cell, which is kept, and each other
    auto fetch = [&](const double *src, double(&x)[K]) __attribute__((always_inline)) {
        double v[K];
#pragma unroll
        for (int m = 0; m < K; ++m) v[m] = src[min(max(rbase + m * 64 + lane, (int64_t)0), n - 1)];
#pragma unroll
        for (int m = 0; m < K; ++m) stage[pos(m * 64 + lane)] = v[m];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < K; ++k) x[k] = stage[lane * (K + 1) + k];
    };
    double va[K], vb[K];
    // B's interior is written before it is read when the pass starts with B:
    // only its ends matter
    const double b0 = a.bfix[0], b1 = a.bfix[n - 1];
    fetch(a.ain, va);
    if (a.phase) {
        __syncthreads();
        fetch(a.bin, vb);
    } else {
#pragma unroll
        for (int k = 0; k < K; ++k) vb[k] = g0 + k <= 0 ? b0 : g0 + k >= n - 1 ? b1 : 0.0;
    }
    // The ends of the array keep their values.  They fall in this region only
    // for the first and last workgroups, as the first and the last point of a
    // lane's run where the region is placed for that: two selects per
    // half-step.  Otherwise every point takes one (a select per point doubles
    // the half-step, and with it a pass whose waves all run at once).
    const bool edge = rbase <= 0 || rbase + R - 1 >= n - 1;
    const bool aligned = a.align && (rbase > 0 || rbase % K == 0) && (rbase + R < n || (n - rbase) % K == 0);
    uint64_t keep[K];
    if (edge) {
#pragma unroll
        for (int k = 0; k < K; ++k) keep[k] = __builtin_amdgcn_ballot_w64(g0 + k == 0 || g0 + k == n - 1);
    }
    // PLAIN: no end in the region; ENDS: at the first or last point of a run
    enum { PLAIN, ENDS, ANY };
    auto half = [&](double(&d)[K], const double(&s)[K], auto mode) __attribute__((always_inline)) {
        constexpr int M = decltype(mode)::value;
        const double left = from_lower(s[K - 1]);
        const double right = from_upper(s[0]);
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const double l = k == 0 ? left : s[k > 0 ? k - 1 : 0];
            const double r = k == K - 1 ? right : s[k < K - 1 ? k + 1 : k];
            const double nv = kW1 * ((l + s[k]) + r);
            if constexpr (M == ANY) d[k] = j_keep(keep[k], nv, d[k]);
            else if constexpr (M == ENDS) d[k] = k == 0 || k == K - 1 ? j_keep(keep[k], nv, d[k]) : nv;
            else d[k] = nv;
        }
    };
    auto steps = [&](auto mode) __attribute__((always_inline)) {
        int s = 0;
        if (a.phase && a.nhalf > 0) {
            half(va, vb, mode);
            s = 1;
        }
        for (; s + 2 <= a.nhalf; s += 2) {
            half(vb, va, mode);
            half(va, vb, mode);
        }
        if (s < a.nhalf) half(vb, va, mode);
    };
    if (!edge) steps(std::integral_constant<int, PLAIN>{});
    else if (aligned) steps(std::integral_constant<int, ENDS>{});
    else steps(std::integral_constant<int, ANY>{});

    // write the tile: A, then (if it is needed) B, each through the LDS
    // transpose
    const int nout = a.write_b ? 2 : 1;
    for (int pass = 0; pass < nout; ++pass) {
        __syncthreads();
#pragma unroll
        for (int k = 0; k < K; ++k) stage[lane * (K + 1) + k] = pass == 0 ? va[k] : vb[k];
        __syncthreads();
        double *out = pass == 0 ? a.aout : a.bout;
        const int64_t lo = pass == 1 && a.write_b == 2 ? 1 : 0, hi = pass == 1 && a.write_b == 2 ? n - 1 : n;
#pragma unroll
        for (int m = 0; m < K; ++m) {
            const int i = m * 64 + lane;
            const int64_t g = rbase + i;
            if (g >= max(own0, lo) && g < min(own0 + a.inner, hi)) out[g] = stage[pos(i)];
        }
    }
}

// ---------------------------------------------------------------- jacobi_2d
// 16 waves per workgroup; wave w owns region rows [w*RPL, (w+1)*RPL) and lane
// l the columns 2l and 2l+1, so the region is (16*RPL) x 128 cells.  West and
// east neighbours across lanes come from DPP shifts, the rows above and below
// a wave's band from the neighbouring waves through LDS (two slots, so one
// barrier per half-step suffices).
// Loads read clamped rows and columns, so they need no guard: as in the row
// march below, a value read for a cell outside the array only feeds boundary
// cells, which are kept, or other cells outside.
// Workgroups whose region holds a boundary cell of the array (uniform) run a
// masked copy of the update, in which a boundary cell keeps the value its
// array had one iteration ago, already in the register it is written to; the
// others carry no mask.
// Bound by FP64 issue (5 operations and two DPP moves per cell) on the
// recomputed halo, then by the launch, loads and stores (about 4 us of a pass):
// 1300^2 with 12 half-steps per pass takes 18.3 us per pass; one masked form
// for every tile, 8 waves of 8 rows per lane, took 22.4.
template <int RPL>
__global__ void __launch_bounds__(1024, RPL <= 4 ? 8 : 4) j2_kernel(J2Args a) {
    constexpr int VEC = 2, W = 16;
    constexpr int R = W * RPL, C = 64 * VEC;
    __shared__ double xch[2][W][2][C];
    // the wave index is uniform over a wave: say so, so that everything that
    // depends only on the row (bounds, masks, row addresses) stays scalar
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // tiles run column by column, so a tile's upper and lower neighbours
    // (whose halos it shares, the larger overlap) are recent in the same L2
    const int b = j_xcd_remap(blockIdx.x, gridDim.x);
    const int tr = b % a.tiles_r, tc = b / a.tiles_r;
    const int64_t n0 = a.n0;
    const int n1 = (int)a.n1;  // < 2^30, checked by the host
    const int ri0 = wave * RPL;
    const int64_t gr0 = (int64_t)tr * a.inner_r - a.hh;  // global row of the region's first row
    const int gc0 = tc * a.inner_c - a.hh;               // and column
    const int64_t gr = gr0 + ri0;                        // global row of r = 0
    const int gc = gc0 + lane * VEC;                     // global column of v = 0
    const bool edge = gr0 <= 0 || gr0 + R >= n0 || gc0 <= 0 || gc0 + C >= n1;  // uniform over the workgroup

    uint64_t colfix[VEC];  // lanes whose column v is a boundary column of the array
#pragma unroll
    for (int v = 0; v < VEC; ++v) colfix[v] = __builtin_amdgcn_ballot_w64(gc + v == 0 || gc + v == n1 - 1);
    auto load = [&](const double *base, double(&x)[RPL][VEC]) __attribute__((always_inline)) {
        const int c0 = min(max(gc, 0), n1 - 1), c1 = min(max(gc + 1, 0), n1 - 1), cp = min(max(gc, 0), n1 - 2);
        auto row = [&](int r) { return base + min(max(gr + r, (int64_t)0), n0 - 1) * n1; };
        if (a.vec16) {
#pragma unroll
            for (int r = 0; r < RPL; ++r) {
                const double2 y = *reinterpret_cast<const double2 *>(row(r) + cp);
                x[r][0] = y.x;
                x[r][1] = y.y;
            }
        } else {
#pragma unroll
            for (int r = 0; r < RPL; ++r) {
                x[r][0] = row(r)[c0];
                x[r][1] = row(r)[c1];
            }
        }
    };
    auto body = [&](auto masked) __attribute__((always_inline)) {
        double va[RPL][VEC], vb[RPL][VEC];
        load(a.ain, va);
        // B: its own values when the pass starts with A, else only the boundary
        // cells count (its interior is written before it is read).  A wave without
        // a boundary row reads one cell a row, the end its lane may hold: on a narrow
        // array most tiles hold some, and reading their whole rows cost them another
        // array's traffic (20000 x 600, 2 half-steps per pass: 1133 us, 929 so).  Two
        // cells a row in every wave cost the others their loads' latency (601 steps of
        // 682 x 6005 3.79 ms, 3.69 so; 300 of 1300^2 916 us, 903).
        if (a.phase) {
            load(a.bin, vb);
        } else if constexpr (decltype(masked)::value) {
            if (gr <= 0 || gr + RPL >= n0) {
                load(a.bfix, vb);
            } else {  // (a lane holds one end at most: three columns or more)
                const double *rb = a.bfix + gr * n1 + (gc <= 0 ? 0 : n1 - 1);
#pragma unroll
                for (int r = 0; r < RPL; ++r) vb[r][0] = vb[r][1] = rb[(int64_t)r * n1];
            }
        } else {
#pragma unroll
            for (int r = 0; r < RPL; ++r) vb[r][0] = vb[r][1] = 0.0;
        }

        int slot = 0;
        auto half = [&](double(&d)[RPL][VEC], const double(&s)[RPL][VEC]) __attribute__((always_inline)) {
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                xch[slot][wave][0][lane * VEC + v] = s[0][v];
                xch[slot][wave][1][lane * VEC + v] = s[RPL - 1][v];
            }
            __syncthreads();
            const int wu = wave > 0 ? wave - 1 : 0, wd = wave < W - 1 ? wave + 1 : wave;
            double up0[VEC], dn0[VEC];
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                // the first and last waves read a slot of their own; the values
                // only feed the region's edge rows
                up0[v] = xch[slot][wu][1][lane * VEC + v];
                dn0[v] = xch[slot][wd][0][lane * VEC + v];
            }
            slot ^= 1;
#pragma unroll
            for (int r = 0; r < RPL; ++r) {
                const double wl = from_lower(s[r][VEC - 1]);
                const double er = from_upper(s[r][0]);
#pragma unroll
                for (int v = 0; v < VEC; ++v) {
                    const double c = s[r][v];
                    const double w = v == 0 ? wl : s[r][v > 0 ? v - 1 : 0];
                    const double e = v == VEC - 1 ? er : s[r][v < VEC - 1 ? v + 1 : v];
                    const double so = r == RPL - 1 ? dn0[v] : s[r < RPL - 1 ? r + 1 : r][v];
                    const double no = r == 0 ? up0[v] : s[r > 0 ? r - 1 : 0][v];
                    const double nv = kW2 * ((((c + w) + e) + so) + no);
                    if constexpr (decltype(masked)::value) {
                        const int64_t i = gr + r;
                        const uint64_t keep = (i == 0 || i == n0 - 1) ? ~(uint64_t)0 : colfix[v];
                        d[r][v] = j_keep(keep, nv, d[r][v]);
                    } else {
                        d[r][v] = nv;
                    }
                }
            }
        };
        int s = 0;
        if (a.phase && a.nhalf > 0) {
            half(va, vb);
            s = 1;
        }
        for (; s + 2 <= a.nhalf; s += 2) {
            half(vb, va);
            half(va, vb);
        }
        if (s < a.nhalf) half(vb, va);

#pragma unroll
        for (int r = 0; r < RPL; ++r) {
            const int ri = ri0 + r;
            const int64_t i = gr + r;
            if (ri < a.hh || ri >= R - a.hh || i >= n0) continue;  // (i >= 0 from ri >= hh)
            double *rowa = a.aout + i * n1;
            double *rowb = a.bout + i * n1;
            const bool binterior_row = i >= 1 && i <= n0 - 2;
            // with vec16 both columns are inside the tile or neither (hh even)
            if (a.vec16 && lane * VEC >= a.hh && lane * VEC < C - a.hh && gc < n1) {
                *reinterpret_cast<double2 *>(rowa + (unsigned)gc) = double2{va[r][0], va[r][1]};
                if (a.write_b == 1) *reinterpret_cast<double2 *>(rowb + (unsigned)gc) = double2{vb[r][0], vb[r][1]};
            }
            if (a.vec16 && a.write_b != 2) continue;
#pragma unroll
            for (int v = 0; v < VEC; ++v) {
                const int ci = lane * VEC + v;
                if (ci < a.hh || ci >= C - a.hh || gc + v >= n1) continue;
                const unsigned j = (unsigned)(gc + v);
                if (!a.vec16) rowa[j] = va[r][v];
                if ((a.write_b == 1 && !a.vec16) ||
                    (a.write_b == 2 && binterior_row && j >= 1 && j <= (unsigned)(n1 - 2)))
                    rowb[j] = vb[r][v];
            }
        }
    };
    if (edge) body(std::true_type{});
    else body(std::false_type{});
}

// ------------------------------------------- jacobi_2d, marching down rows
// The form for large arrays.  A workgroup is one wave and owns a strip of 128
// columns (two per lane; the first and last hh are halo, recomputed) and a
// segment of rows, and marches down the rows applying NH half-steps in one
// pass: at step q, level s (the arrays after s half-steps; odd levels are B,
// even levels A) is computed for row q - s + 1, from level s - 1 of rows
// q - s .. q - s + 2, the last of which level s - 1 has just computed.  For
// every level each lane keeps three rows of its columns in registers, so the
// rows above and below come from the lane itself and the columns left and
// right from the adjacent lanes (DPP): no LDS and no barrier.  Row x of every
// level lives in register slot x mod 3; the loop is unrolled three times, so
// the slots are fixed at compile time and no register is copied as the march
// advances.  Compared with the region tiles above, only the columns carry a
// halo, and the rows before a segment are recomputed once (NH - 1 rows per
// level; a level computes its rows from the first step on, the ones it cannot
// know yet are never read by a row that counts).
// Loads of level 0 are issued three rows ahead of use.  They read clamped rows
// and columns, so they need no guard: a value read for a row or column
// outside the array only ever feeds a boundary cell of the array, which is
// replaced by its fixed value (a select, so whatever was computed there is
// dropped), or another cell outside the array.
// The array's boundary cells keep their values at every level: level s takes
// them from level s - 2 (the same array; the slot it is about to leave behind
// still holds that row), level 1 from B in memory.  A wave that holds no
// boundary cell skips all of this.  Requires hh even.
// What bounds it: FP64 issue (5 operations per cell and four 32-bit DPP moves
// per pair, on 128 / (128 - 2 hh) of the columns), then memory: 23400^2 with
// 16 half-steps takes 183 us per half-step; the same kernel without loads and
// stores 146, a copy of the array once per pass about 90.  Two columns per
// lane leave the registers for rows fetched three ahead and 16 half-steps per
// pass.  Four columns per lane need fewer moves per cell, but fit only 8
// half-steps with rows fetched one ahead, and waited on memory: 266 us per
// half-step, 254 with the boundary selects taken out.
typedef double j2m_v2 __attribute__((ext_vector_type(2), aligned(8)));  // rows of any length

struct J2MArgs {
    const double *ain, *bfix;  // level 0 (A); B's values (its boundary cells never change)
    double *aout, *bout;
    int64_t n0, n1;
    int hh, strips, segs, seg_rows, write_b;
};

// Strip and segment of a workgroup.  The waves that hold boundary cells run
// longer (selects at every level), so they go first: the first and last
// segment, then the first strip and the last two on the other segments; the
// rest fill the GPU evenly behind them.  The rest run strips fastest within
// an XCD's share, so that neighbours share their halo columns in its L2.
__device__ __forceinline__ void j2m_tile(int strips, int segs, int &strip, int &seg) {
    const int b = blockIdx.x;
    if (strips < 4 || segs < 3) {
        const int t = j_xcd_remap(b, gridDim.x);
        strip = t % strips;
        seg = t / strips;
        return;
    }
    const int rows = 2 * strips, first = rows + 3 * (segs - 2);
    if (b < rows) {
        seg = b < strips ? 0 : segs - 1;
        strip = b < strips ? b : b - strips;
    } else if (b < first) {
        const int t = b - rows;
        seg = 1 + t / 3;
        strip = t % 3 == 0 ? 0 : strips - (t % 3);
    } else {
        const int t = j_xcd_remap(b - first, (int)gridDim.x - first);
        seg = 1 + t / (strips - 3);
        strip = 1 + t % (strips - 3);
    }
}

template <int NH>
__global__ void __launch_bounds__(64) j2m_kernel(J2MArgs a) {
    constexpr int CPL = 2, C = 64 * CPL, D = 3;  // columns per lane and strip, rows fetched ahead
    const int lane = threadIdx.x;
    int strip, seg;
    j2m_tile(a.strips, a.segs, strip, seg);
    const int n0 = (int)a.n0;  // < 2^30, checked by the host (so are the row indices below)
    const int n1 = (int)a.n1;
    const int ci = CPL * lane;                           // column offset in the strip
    const int gc = strip * (C - 2 * a.hh) - a.hh + ci;   // column of this lane's first value (even)
    // the lane's load column, clamped into the array, and whether this strip
    // stores its columns; with an odd n1 the last column is the first of a
    // lane's two (`last`: it loads them one column early and stores one)
    const int col = min(max(gc, 0), n1 - 2);
    const bool own = gc >= 0 && gc < n1 && ci >= a.hh && ci < C - a.hh;
    const bool last = gc == n1 - 1;
    // lanes whose first column is 0 or n1 - 1, whose second is n1 - 1
    const uint64_t keep[CPL] = {__builtin_amdgcn_ballot_w64(gc == 0 || last), __builtin_amdgcn_ballot_w64(gc == n1 - 2)};
    const bool edge = (keep[0] | keep[1]) != 0;  // uniform over the wave
    const int R0 = seg * a.seg_rows;
    const int R1 = min(n0, R0 + a.seg_rows);
    const bool rowedge = R0 - NH <= 0 || R1 + NH > n0 - 1;  // rows in flight include a boundary row
    if (R0 >= R1) return;  // a segment past the last row

    auto load_row = [&](const double *base, int r, double (&x)[CPL]) {  // the row clamped into the array
        const double *rp = base + (int64_t)min(max(r, 0), n0 - 1) * n1;
        const j2m_v2 v = *reinterpret_cast<const j2m_v2 *>(rp + col);
        x[0] = v.x;
        x[1] = v.y;
    };
    // the column a `last` lane needs is the second of the pair it loaded
    auto fix_last = [&](double (&x)[CPL]) { x[0] = last ? x[1] : x[0]; };

    double S[NH][3][CPL];  // [level][row slot: row mod 3, counted from q0][column]
    double P[D][CPL];      // level-0 rows in flight
    double PB[D][CPL];     // B on the same rows, two back (waves with a boundary cell)
    const int q0 = R0 - NH + 1, qlast = R1 + NH - 2;
#pragma unroll
    for (int s = 1; s < NH; ++s)
#pragma unroll
        for (int j = 0; j < 3; ++j)
#pragma unroll
            for (int k = 0; k < CPL; ++k) S[s][j][k] = 0.0;
    // level 0: rows q0 - 1 and q0 now, rows q0 + 1 .. q0 + D in flight
    load_row(a.ain, q0 - 1, S[0][2]);
    load_row(a.ain, q0, S[0][0]);
    fix_last(S[0][2]);
    fix_last(S[0][0]);
    const bool general_wave = edge || rowedge;
#pragma unroll
    for (int d = 0; d < D; ++d) {
        load_row(a.ain, q0 + 1 + d, P[(1 + d) % D]);
        PB[d][0] = PB[d][1] = 0.0;
        if (general_wave) load_row(a.bfix, q0 + d, PB[d]);
    }

    // Step q at phase PH = (q - q0) mod 3.  GENERAL: the wave holds boundary
    // cells; the plain form drops the checks and selects.
    auto step = [&](int q, auto PH, auto GENERAL) __attribute__((always_inline)) {
        constexpr int ph = decltype(PH)::value;
        constexpr bool general = decltype(GENERAL)::value;
        // level 0 takes row q + 1; row q + 1 + D is fetched into its place
        double(&l0)[CPL] = S[0][(ph + 1) % 3];
        double(&pf)[CPL] = P[(ph + 1) % D];
#pragma unroll
        for (int k = 0; k < CPL; ++k) l0[k] = pf[k];
        if constexpr (general) fix_last(l0);
        load_row(a.ain, q + 1 + D, pf);
#pragma unroll
        for (int s = 1; s <= NH; ++s) {
            const int r = q - s + 1;
            // level s - 1 rows r - 1, r, r + 1 and the slot of row r
            const int lo = ((ph - s) % 3 + 3) % 3, mid = ((ph - s + 1) % 3 + 3) % 3,
                      hi = ((ph - s + 2) % 3 + 3) % 3;
            const double(&in0)[CPL] = S[s - 1][lo];
            const double(&in1)[CPL] = S[s - 1][mid];
            const double(&in2)[CPL] = S[s - 1][hi];
            const double wl = from_lower(in1[CPL - 1]);
            const double er = from_upper(in1[0]);
            double nv[CPL];
#pragma unroll
            for (int k = 0; k < CPL; ++k) {
                const double w = k ? in1[k - 1] : wl;
                const double e = k < CPL - 1 ? in1[k + 1] : er;
                nv[k] = kW2 * ((((in1[k] + w) + e) + in2[k]) + in0[k]);
            }
            if constexpr (general) {
                // boundary cells of row r keep their values: those of level
                // s - 2 (level 0 and up), of B in memory (level 1)
                if (s == 1) fix_last(PB[ph]);
                const double(&old)[CPL] = s == 1 ? PB[ph] : S[s >= 2 ? s - 2 : 0][mid];
                const bool frow = r == 0 || r == n0 - 1;  // uniform: the whole row
#pragma unroll
                for (int k = 0; k < CPL; ++k) nv[k] = j_keep(frow ? ~(uint64_t)0 : keep[k], nv[k], old[k]);
            }
            if (s < NH) {
#pragma unroll
                for (int k = 0; k < CPL; ++k) S[s][mid][k] = nv[k];
            }
            // A's row r is stored where it belongs to the segment, B's row
            // (the level before) by the last pass only; a store covers whole
            // lines and goes out with the streaming hint
            if (s == NH && r >= R0 && own) {
                double *o = a.aout + (int64_t)r * n1 + gc;
                if (general && last) *o = nv[0];
                else __builtin_nontemporal_store(j2m_v2{nv[0], nv[1]}, reinterpret_cast<j2m_v2 *>(o));
            }
            if (s == NH - 1 && a.write_b != 0 && r >= R0 && r < R1 && own) {
                double *o = a.bout + (int64_t)r * n1 + gc;
                if (a.write_b == 1) {
                    if (general && last) *o = nv[0];
                    else __builtin_nontemporal_store(j2m_v2{nv[0], nv[1]}, reinterpret_cast<j2m_v2 *>(o));
                } else if (r >= 1 && r <= n0 - 2) {  // B's interior only
                    if (gc >= 1 && !last) o[0] = nv[0];
                    if (gc + 1 <= n1 - 2) o[1] = nv[1];
                }
            }
        }
        if constexpr (general) load_row(a.bfix, q + D, PB[ph]);
    };
    using P0 = std::integral_constant<int, 0>;
    using P1 = std::integral_constant<int, 1>;
    using P2 = std::integral_constant<int, 2>;
    // The loop runs whole groups of three and the last one or two steps
    // follow it, so every register keeps its place across the loop's back
    // edge (a copy there would wait for the rows still in flight).
    auto march = [&](auto GENERAL) __attribute__((always_inline)) {
        int q = q0;
        for (; q + 2 <= qlast; q += 3) {
            step(q, P0{}, GENERAL);
            step(q + 1, P1{}, GENERAL);
            step(q + 2, P2{}, GENERAL);
        }
        if (q <= qlast) step(q, P0{}, GENERAL);
        if (q + 1 <= qlast) step(q + 1, P1{}, GENERAL);
    };
    if (general_wave) march(std::true_type{});
    else march(std::false_type{});
}

// ------------------------------------------------------------- host side
constexpr int kJ2C = 128;  // region columns (2D)
constexpr int kJ1MaxTb = 256, kJ2MaxTb = 16;
constexpr size_t kJAlign = 256;

// Points per lane in 1D.  Runs of 16 cost the fewest cross-lane moves per
// point without spilling (runs of 32 measured slower); they are used when the
// array gives at least 2048 workgroups with them.  Smaller arrays take the
// shortest admissible run (tile at least half the region), spreading the
// work over more CUs.  DCP_J1_K forces a length (tuning runs only).
// Halo of a region placed by the array's ends (see j1_kernel): whole runs, with
// room to move the region by less than one.
int64_t j1_halo(int64_t K, int64_t hh) { return (hh + 2 * (K - 1)) / K * K; }

int j1_pick_k(int64_t n, int64_t hh) {
    auto admissible = [&](int k) { return 64 * k - 2 * hh >= 32 * k; };
    const char *forced = dcp::tuning_env("DCP_J1_K");
    if (forced && *forced) {
        const int k = std::atoi(forced);
        if ((k == 4 || k == 8 || k == 16 || k == 32) && 64 * k > 2 * hh) return k;
    }
    if (admissible(16) && (n + (64 * 16 - 2 * hh) - 1) / (64 * 16 - 2 * hh) >= 2048) return 16;
    for (int k : {4, 8, 16, 32})
        if (admissible(k)) return k;
    return 32;
}

// Rows per lane of the 2D region tiles (16 waves, so 32 to 128 rows of 128
// columns): the least time by a price for a tile and for the tiles of one CU,
// fitted to 111 arrays of 100 to 20,000 rows and columns with 1, 4, 8 and 12
// half-steps per pass (most of them narrow), where its choice takes 1.000 to 1.005
// times the fastest in the mean, at most 1.07.  A tile takes 1 + rows per lane *
// (1.25 + 0.04 * half-steps), whether it holds boundary cells or not.  Tiles of up
// to four rows per lane (64 VGPRs) run two to a CU and hide each other's waits: each
// beyond the CU's first adds half a tile's time (48 to 52%).  Taller ones run one by
// one.  us per pass, in runs of 8 (118 x 9505) and 12 half-steps: 118 x 9505 11.9 with
// four rows per lane, 14.7 with two; 200 x 3000 12.7 with four, 17.1 with six; 300^2
// 8.1 with two, 12.0 with four; 1300^2 18.3 with six (247 tiles), 19.5 with four
// (429); 2000^2 33 with four, 39 with seven.  DCP_J2_CFG = 0, 1 or 2 forces 4, 6 or 8
// rows per lane where the halo leaves a tile (tuning runs only).
int j2_pick_rpl(int64_t n0, int64_t n1, int64_t hh) {
    const char *fc = dcp::tuning_env("DCP_J2_CFG");
    if (fc && *fc) {
        const int c = std::atoi(fc);
        if (c >= 0 && c < 3 && 16 * (4 + 2 * c) > 2 * hh) return 4 + 2 * c;
    }
    int best = 8;
    double cost = 1e300;
    for (int rpl = 2; rpl <= 8; ++rpl) {
        const int64_t rows = 16 * rpl, inner_r = rows - 2 * hh, inner_c = kJ2C - 2 * hh;
        if (inner_r <= 0) continue;
        const double tiles = (double)((n0 + inner_r - 1) / inner_r) * (double)((n1 + inner_c - 1) / inner_c);
        const double per_cu = std::ceil(tiles / 256.0), tile = 1.0 + rpl * (1.25 + 0.04 * (double)hh);
        const double x = rpl <= 4 ? tile * (1.0 + (0.44 + 0.02 * rpl) * (per_cu - 1.0))
                                  : tile * 0.5 * (per_cu + std::max(1.0, tiles / 256.0));
        if (x < cost) {
            cost = x;
            best = rpl;
        }
    }
    return best;
}

// The row-marching form (j2m_kernel): used for arrays that give it at least
// 1900 waves (nearly two per SIMD) with row segments of at least 4*NH rows; passes of
// 4 to 16 half-steps (even) that start with B (whole time-loop iterations).  More, shorter
// segments even out the end of a pass (a share of about 2048 / waves of it)
// but recompute 2*NH rows each; their sum is least near
// sqrt(768 * n0 * strips / NH) waves.  Measured with 16 half-steps, us per
// half-step with 4096 / 8192 / 16384 / 24576 waves: 46800^2 906 / 807 / 736 /
// 720 (the rule gives 33,000), 23400^2 221 / 194 / 183 / 186 (16,500),
// 12000^2 54 / 52 / 55 / 58 (8,500).  Below the 1900 waves the region tiles
// are as fast: 3000^2 5.4-6.1 against 5.6 us (3500^2, 1998 waves, 7.9 against 5.8).
// Passes of up to 10 half-steps march from 2^24 elements on, where the array read and
// the one written no longer fit the 256 MB cache, from which the tiles' halos come.
// 200 half-steps, ms, tiles / march, in passes of 4: 3000^2 1.55 / 2.16, 4000^2 2.58 /
// 3.46, 4500^2 4.06 / 4.02, 5500^2 6.33 / 5.87; of 8: 1.02 / 1.12, 1.71 / 1.79, 2.32 /
// 2.24, 3.55 / 3.48; of 12: 1.02 / 1.04, 1.76 / 1.74, 2.26 / 1.95, 3.44 / 2.82.
// DCP_J2_MODE = 3 forces the form where it applies, 1 or 2 the region tiles (tuning
// runs only).
struct J2MPlan {
    bool use = false;
    int strips = 0, segs = 0, seg_rows = 0;
};

J2MPlan j2m_pick(int64_t n0, int64_t n1, int64_t hh) {
    J2MPlan m;
    constexpr int64_t C = 128;
    if (n0 < 3 || n1 < 3 || n0 >= ((int64_t)1 << 30) || hh % 2 != 0 || hh < 4 || hh > 16)
        return m;
    const int64_t strips = (n1 + (C - 2 * hh) - 1) / (C - 2 * hh);
    const int64_t maxsegs = std::max<int64_t>(1, n0 / (4 * hh));
    const int64_t want = (int64_t)std::sqrt(768.0 * (double)n0 * (double)strips / (double)hh);
    const int64_t segs = std::max<int64_t>(1, std::min<int64_t>(maxsegs, (want + strips - 1) / strips));
    if (strips * segs > INT32_MAX / 2) return m;
    m.seg_rows = (int)((n0 + segs - 1) / segs);
    m.segs = (int)((n0 + m.seg_rows - 1) / m.seg_rows);
    m.strips = (int)strips;
    m.use = (int64_t)m.strips * m.segs >= 1900 && (hh > 10 || n0 * n1 >= ((int64_t)1 << 24));
    const char *fm = dcp::tuning_env("DCP_J2_MODE");
    if (fm && *fm) m.use = std::atoi(fm) == 3;
    return m;
}

template <int K>
hipError_t j1_launch(int64_t blocks, const J1Args &a, hipStream_t sm) {
    hipLaunchKernelGGL(j1_kernel<K>, dim3((unsigned)blocks), dim3(64), 0, sm, a);
    return hipGetLastError();
}

size_t j_align(size_t x) { return (x + kJAlign - 1) / kJAlign * kJAlign; }

bool j_overlaps(const void *a, size_t na, const void *b, size_t nb) {
    if (!a || !b || na == 0 || nb == 0) return false;
    const uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
    return a0 < b0 + nb && b0 < a0 + na;
}

struct JGeo {
    int dims = 1;
    int64_t n0 = 0, n1 = 1, count = 0;
    bool has_interior = false;
};

int j_geo(int dims, int64_t n0, int64_t n1, JGeo *g) {
    if (dims != 1 && dims != 2) return DCP_E_ARG;
    if (n0 < 0 || (dims == 2 && n1 < 0)) return DCP_E_SHAPE;
    const int64_t lim = ((int64_t)1 << 60) / 8;
    g->dims = dims;
    g->n0 = n0;
    g->n1 = dims == 2 ? n1 : 1;
    if (dims == 2 && n1 > 0 && n0 > lim / n1) return DCP_E_SHAPE;
    if (dims == 2 && n1 >= ((int64_t)1 << 30)) return DCP_E_SHAPE;
    if (n0 > lim) return DCP_E_SHAPE;
    g->count = n0 * g->n1;
    g->has_interior = dims == 1 ? n0 >= 3 : (n0 >= 3 && n1 >= 3);
    return DCP_OK;
}

// Half-steps per pass.  The defaults are the measured best on MI355X: in 1D
// 64 for small arrays (the pass count is launch-bound) and 128 for large
// ones; in 2D 16 where the row-marching form applies (23400^2, us per
// half-step with 8 / 10 / 12 / 14 / 16: 236 / 209 / 187 / 185 / 183), else 12
// (10-14 measured within a few percent with the region tiles at 1300^2).
int j_tblock(const JGeo &g, int32_t tblock, int *hp) {
    const int mx = g.dims == 1 ? kJ1MaxTb : kJ2MaxTb;
    if (tblock < 0 || tblock > mx) return DCP_E_ARG;
    if (tblock > 0) *hp = tblock;
    else if (g.dims == 1) *hp = g.count >= ((int64_t)1 << 22) ? 128 : 64;
    else *hp = j2m_pick(g.n0, g.n1, 16).use ? 16 : 12;
    return DCP_OK;
}

// The pass schedule.  Passes alternate between the caller's arrays and the
// workspace copies, and their number is even so the result ends in the
// caller's arrays.  When every pass can hold a whole number of time-loop
// iterations (an even number of half-steps), every pass starts by writing B
// from A, so B's interior is never read across a pass boundary: only the last
// pass stores B, and B's boundary is always read from the caller's B (it
// never changes).  Otherwise (one half-step per pass, or a single iteration)
// passes split at half-steps and store both arrays.
struct JPlan {
    int64_t halves = 0, passes = 0, per = 0, rem = 0, hh = 0;
    bool whole = false;  // pass sizes counted in iterations (2 half-steps each)
    int64_t size(int64_t i) const {
        const int64_t s = per + (i < rem ? 1 : 0);
        return whole ? 2 * s : s;
    }
};

JPlan j_plan(const JGeo &g, int32_t tsteps, int hp) {
    JPlan p;
    if (tsteps <= 1 || !g.has_interior) return p;
    const int64_t iters = (int64_t)tsteps - 1;
    p.halves = 2 * iters;
    if (hp >= 2) {
        int64_t P = (iters + hp / 2 - 1) / (hp / 2);
        if (P & 1) ++P;
        if (P <= iters) {
            p.whole = true;
            p.passes = P;
            p.per = iters / P;
            p.rem = iters % P;
            p.hh = 2 * (p.per + (p.rem ? 1 : 0));
            return p;
        }
    }
    int64_t P = (p.halves + hp - 1) / hp;
    if (P & 1) ++P;
    p.passes = P;
    p.per = p.halves / P;
    p.rem = p.halves % P;
    p.hh = p.per + (p.rem ? 1 : 0);
    return p;
}

size_t j_ws_need(const JGeo &g, const JPlan &p) {
    return p.passes ? 2 * j_align((size_t)g.count * sizeof(double)) : 0;
}

int j_check_buffers(const JGeo &g, const double *A, const double *B, const void *ws, size_t ws_bytes,
                    size_t need) {
    const size_t bytes = (size_t)g.count * sizeof(double);
    if (g.count > 0 && (!A || !B)) return DCP_E_NULL;
    if (j_overlaps(A, bytes, B, bytes)) return DCP_E_ALIAS;
    if (need) {
        if (ws_bytes < need) return DCP_E_WORKSPACE;
        if (!ws) return DCP_E_NULL;
        if (j_overlaps(ws, need, A, bytes) || j_overlaps(ws, need, B, bytes)) return DCP_E_ALIAS;
    }
    return DCP_OK;
}

template <typename Launch>
int j_run_passes(const JGeo &g, const JPlan &p, double *A, double *B, void *ws, Launch launch) {
    const size_t fb = j_align((size_t)g.count * sizeof(double));
    double *WA = reinterpret_cast<double *>(static_cast<char *>(ws));
    double *WB = reinterpret_cast<double *>(static_cast<char *>(ws) + fb);
    int64_t done = 0;
    for (int64_t i = 0; i < p.passes; ++i) {
        const int nh = (int)p.size(i);
        const bool even = (i & 1) == 0;
        const double *ain = even ? A : WA;
        const double *bin = even ? B : WB;
        double *aout = even ? WA : A;
        double *bout = even ? WB : B;
        const bool last = i == p.passes - 1;
        const int write_b = p.whole ? (last ? 2 : 0) : 1;
        const double *bfix = p.whole ? B : bin;
        if (launch(ain, bin, bfix, aout, bout, nh, (int)(done & 1), write_b) != hipSuccess) return DCP_E_HIP;
        done += nh;
    }
    return DCP_OK;
}

}  // namespace

extern "C" {

int dcp_jacobi_workspace_bytes(int dims, int64_t n0, int64_t n1, int32_t tsteps, int32_t tblock,
                               size_t *bytes) {
    if (!bytes) return DCP_E_NULL;
    JGeo g;
    int st = j_geo(dims, n0, n1, &g);
    if (st != DCP_OK) return st;
    int hp = 0;
    st = j_tblock(g, tblock, &hp);
    if (st != DCP_OK) return st;
    *bytes = j_ws_need(g, j_plan(g, tsteps, hp));
    return DCP_OK;
}

int dcp_jacobi_plan(int dims, int64_t n0, int64_t n1, int32_t tsteps, int32_t tblock, int64_t *passes,
                    int32_t *halo) {
    if (!passes || !halo) return DCP_E_NULL;
    JGeo g;
    int st = j_geo(dims, n0, n1, &g);
    if (st != DCP_OK) return st;
    int hp = 0;
    st = j_tblock(g, tblock, &hp);
    if (st != DCP_OK) return st;
    const JPlan p = j_plan(g, tsteps, hp);
    *passes = p.passes;
    *halo = (int32_t)p.hh;
    return DCP_OK;
}

int dcp_jacobi_1d(int32_t tsteps, double *A, double *B, int64_t n, int32_t tblock, void *ws, size_t ws_bytes,
                  void *stream) {
    JGeo g;
    int st = j_geo(1, n, 1, &g);
    if (st != DCP_OK) return st;
    int hp = 0;
    st = j_tblock(g, tblock, &hp);
    if (st != DCP_OK) return st;
    const JPlan p = j_plan(g, tsteps, hp);
    st = j_check_buffers(g, A, B, ws, ws_bytes, j_ws_need(g, p));
    if (st != DCP_OK || p.passes == 0) return st;
    const int K = j1_pick_k(n, p.hh);
    // the wider halo costs about 6% more waves: worth it while they run at once
    // (T = 1000, n = 24,000: 209 us with a select per point at the ends, 177
    // with two; n = 300,001: 323 and 310; n = 10^6: 655 and 674)
    const bool align = K <= 8 && 64 * K > 2 * j1_halo(K, p.hh) && n / (64 * K - 2 * p.hh) < 4096;
    const int64_t hr = align ? j1_halo(K, p.hh) : p.hh, inner = 64 * K - 2 * hr;
    const int64_t blocks = (n + inner - 1) / inner;
    if (blocks > INT32_MAX) return DCP_E_SHAPE;
    hipStream_t sm = static_cast<hipStream_t>(stream);
    return j_run_passes(g, p, A, B, ws,
                        [&](const double *ain, const double *bin, const double *bfix, double *aout, double *bout,
                            int nh, int ph, int wb) {
                            const J1Args a{ain, bin, bfix, aout, bout, n, inner, (int)hr, nh, ph, wb, align ? 1 : 0};
                            switch (K) {
                                case 4: return j1_launch<4>(blocks, a, sm);
                                case 8: return j1_launch<8>(blocks, a, sm);
                                case 16: return j1_launch<16>(blocks, a, sm);
                                default: return j1_launch<32>(blocks, a, sm);
                            }
                        });
}

int dcp_jacobi_2d(int32_t tsteps, double *A, double *B, int64_t n0, int64_t n1, int32_t tblock, void *ws,
                  size_t ws_bytes, void *stream) {
    JGeo g;
    int st = j_geo(2, n0, n1, &g);
    if (st != DCP_OK) return st;
    int hp = 0;
    st = j_tblock(g, tblock, &hp);
    if (st != DCP_OK) return st;
    const JPlan p = j_plan(g, tsteps, hp);
    st = j_check_buffers(g, A, B, ws, ws_bytes, j_ws_need(g, p));
    if (st != DCP_OK || p.passes == 0) return st;
    const int rpl = j2_pick_rpl(n0, n1, p.hh);
    const int inner_r = 16 * rpl - 2 * (int)p.hh, inner_c = kJ2C - 2 * (int)p.hh;
    const int64_t tiles_r = (n0 + inner_r - 1) / inner_r, tiles_c = (n1 + inner_c - 1) / inner_c;
    if (tiles_c > INT32_MAX || tiles_r > INT32_MAX / tiles_c) return DCP_E_SHAPE;
    hipStream_t sm = static_cast<hipStream_t>(stream);
    auto launch_tiles = [&](const J2Args &a) -> hipError_t {
        const dim3 grid((unsigned)(tiles_r * tiles_c)), block(1024);
        switch (rpl) {
            case 2: hipLaunchKernelGGL(j2_kernel<2>, grid, block, 0, sm, a); break;
            case 3: hipLaunchKernelGGL(j2_kernel<3>, grid, block, 0, sm, a); break;
            case 4: hipLaunchKernelGGL(j2_kernel<4>, grid, block, 0, sm, a); break;
            case 5: hipLaunchKernelGGL(j2_kernel<5>, grid, block, 0, sm, a); break;
            case 6: hipLaunchKernelGGL(j2_kernel<6>, grid, block, 0, sm, a); break;
            case 7: hipLaunchKernelGGL(j2_kernel<7>, grid, block, 0, sm, a); break;
            default: hipLaunchKernelGGL(j2_kernel<8>, grid, block, 0, sm, a); break;
        }
        return hipGetLastError();
    };
    const J2MPlan mp = j2m_pick(n0, n1, p.hh);
    auto launch_march = [&](const J2MArgs &m, int nh) -> hipError_t {
        const dim3 grid((unsigned)((int64_t)mp.strips * mp.segs));
        switch (nh) {
            case 4: hipLaunchKernelGGL(j2m_kernel<4>, grid, dim3(64), 0, sm, m); break;
            case 6: hipLaunchKernelGGL(j2m_kernel<6>, grid, dim3(64), 0, sm, m); break;
            case 8: hipLaunchKernelGGL(j2m_kernel<8>, grid, dim3(64), 0, sm, m); break;
            case 10: hipLaunchKernelGGL(j2m_kernel<10>, grid, dim3(64), 0, sm, m); break;
            case 12: hipLaunchKernelGGL(j2m_kernel<12>, grid, dim3(64), 0, sm, m); break;
            case 14: hipLaunchKernelGGL(j2m_kernel<14>, grid, dim3(64), 0, sm, m); break;
            default: hipLaunchKernelGGL(j2m_kernel<16>, grid, dim3(64), 0, sm, m); break;
        }
        return hipGetLastError();
    };
    return j_run_passes(g, p, A, B, ws,
                        [&](const double *ain, const double *bin, const double *bfix, double *aout, double *bout,
                            int nh, int ph, int wb) {
                            const bool v16 = (n1 % 2 == 0) && (p.hh % 2 == 0) &&
                                             ((uintptr_t)ain | (uintptr_t)bin | (uintptr_t)bfix |
                                              (uintptr_t)aout | (uintptr_t)bout) % 16 == 0;
                            // whole iterations (B first, B's interior not read):
                            // the row-marching form
                            if (mp.use && p.whole && ph == 0 && nh >= 4 && nh <= 16 && nh % 2 == 0) {
                                const J2MArgs m{ain, bfix, aout, bout, n0, n1, (int)p.hh, mp.strips, mp.segs,
                                                mp.seg_rows, wb};
                                return launch_march(m, nh);
                            }
                            const J2Args a{ain, bin, bfix, aout, bout, n0, n1, inner_r, inner_c,
                                           (int)tiles_r, (int)p.hh, nh, ph, wb, v16 ? 1 : 0};
                            return launch_tiles(a);
                        });
}

}  // extern "C"
