// dcp_block.hip -- two or three fused steps per pass on small grids (gfx950).
//
// The marching kernels (dcp_tbk.hip, dcp_tblock.hip) walk up z and wait for
// memory plane by plane; on a grid of a few million points each workgroup has
// only a handful of planes, and those waits are the pass.  Here a workgroup
// takes a block of bx x by x BZ points with a halo of B points on every side,
// issues all its loads at once, applies the B steps and stores the block: one
// wait for memory per pass.
//   * a lane owns one (x, y) column of the block and its halo; the column's
//     FZ = BZ + 2B values sit in registers (the z-neighbours), and each level
//     is published in LDS for the x- and y-neighbours, two barriers per step;
//   * step s is computed on the block plus a halo of B - s points;
//   * the halo is recomputed and reread (about four times the block), which is
//     why larger grids march instead.
// A pass of three steps at 64^3 FP64 takes 10.5 us (14.2 marching): about 4 us
// for the launch and the loads, the rest LDS reads, FP64 issue and the two
// barriers of each step, about 2 us a step with one workgroup per CU.  Run of
// 10 steps with norms 48.1 -> 39.2 us; gradient through 40 steps 381 -> 292 us.
// Every point is computed with the one-step kernel's operations, so a pass
// equals B single steps bit for bit; sums are reduced over the owned points.
#include "dcp_internal.h"

#include <algorithm>

namespace dcp {
namespace {

// Index i (any integer) under the boundary rule on [0, n); -1 = ghost.
template <int BC>
__device__ __forceinline__ int b_wrap(int i, int n) {
    if (i >= 0 && i < n) return i;
    if constexpr (BC == 1) {
        const int m = i % n;
        return m < 0 ? m + n : m;
    }
    return -1;
}

__device__ __forceinline__ int b_xcd_remap(int b, int nb) {
    const int per = nb >> 3, rem = nb & 7;
    const int xcd = b & 7, j = b >> 3;
    return xcd * per + min(xcd, rem) + j;
}

constexpr int kLanes = kBlkLanes;  // at least a column per lane of the block's frame

// OP = SOP_FWD: u = u_t, q[0] = f, out = u_{t+B}, mid[s-1] = u_{t+s} or null;
//   sums of step s: the norms.
// OP = SOP_ADJ (B = 2): u = lambda_{t+1}, q[s-1] = u_{t-s+1}, out =
//   lambda_{t-1}; sums: the parameter sums of steps t and t - 1.
// OP = SOP_ADJL: SOP_ADJ, and lam = (lam + lambda_{t+1}) + lambda_t
//   (lam_first: lam is not read, taken as 0).
template <typename T, int B, int BZ, int BC, int OP, bool RED>
__global__ void __launch_bounds__(kLanes) block_kernel(BlkArgs a) {
    constexpr int FZ = BZ + 2 * B;
    constexpr bool ADJ = OP != SOP_FWD, LAM = OP == SOP_ADJL;
    extern __shared__ __align__(16) unsigned char blk_smem[];
    T *const SM = reinterpret_cast<T *>(blk_smem);  // planes 1 .. FZ-2 of a level
    const int nx = (int)a.nx, ny = (int)a.ny, nz = (int)a.nz;
    const int64_t sz = a.nx * a.ny;
    const int FX = a.bx + 2 * B, FY = a.by + 2 * B, FP = FX * FY;

    const int tid = threadIdx.x;
    const int Lb = b_xcd_remap(blockIdx.x, gridDim.x);
    const int tx = Lb % a.tiles_x, tyz = Lb / a.tiles_x;
    const int x0 = tx * a.bx, y0 = (tyz % a.tiles_y) * a.by, z0 = (tyz / a.tiles_y) * BZ;
    const bool in = tid < FP;
    const int cy = in ? tid / FX : 0, cx = in ? tid % FX : 0;
    const int gx = b_wrap<BC>(x0 - B + cx, nx), gy = b_wrap<BC>(y0 - B + cy, ny);
    const bool ghost = gx < 0 || gy < 0;  // Dirichlet: every level reads 0
    const int col = ghost ? 0 : gy * nx + gx;
    const bool own = in && cx >= B && cx < B + a.bx && cy >= B && cy < B + a.by && x0 + cx - B < nx && y0 + cy - B < ny;
    const T C0 = (T)a.c0, C1 = (T)a.c1, C2 = (T)a.c2;

    // all loads up front, each lane from a valid column of a valid plane
    // (ghosts are zeroed); plane z of the frame is grid plane z0 - B + z
    auto plane = [&](const void *p, int z) -> const T * {
        const int zr = b_wrap<BC>(z0 - B + z, nz);
        return static_cast<const T *>(p) + (int64_t)(zr >= 0 ? zr : 0) * sz;
    };
    T cur[FZ], q1[FZ], q2[ADJ ? FZ : 1], lv[LAM ? BZ : 1];
#pragma unroll
    for (int z = 0; z < FZ; ++z) cur[z] = plane(a.u, z)[col];
#pragma unroll
    for (int z = 1; z < FZ - 1; ++z) q1[z] = plane(a.q[0], z)[col];
    if constexpr (ADJ) {
#pragma unroll
        for (int z = 2; z < FZ - 2; ++z) q2[z] = plane(a.q[1], z)[col];
    }
    if constexpr (LAM) {
#pragma unroll
        for (int z = 0; z < BZ; ++z) lv[z] = T(0);
        // the running sum is read where it is written: another block's points are
        // being changed meanwhile
        if (own && !a.lam_first) {
#pragma unroll
            for (int z = 0; z < BZ; ++z) lv[z] = plane(a.lam, z + B)[col];
        }
    }
    if constexpr (BC == 0) {
#pragma unroll
        for (int z = 0; z < FZ; ++z)
            if (ghost || z0 - B + z < 0 || z0 - B + z >= nz) cur[z] = T(0);
    }

    // LDS places of the x- and y-neighbours; a lane on the frame's edge reads
    // its own (what it computes is not used)
    const int me = in ? tid : 0;
    const int xm = cx > 0 ? me - 1 : me, xp = cx < FX - 1 ? me + 1 : me;
    const int ym = cy > 0 ? me - FX : me, yp = cy < FY - 1 ? me + FX : me;
    double s0[B], s1[B];
#pragma unroll
    for (int s = 0; s < B; ++s) s0[s] = s1[s] = 0.0;
    // The B steps, without branches in a step so that its planes' LDS reads and
    // arithmetic overlap: every lane computes and sums every plane of the
    // level; lanes that own nothing drop their sums at the end.
#pragma unroll
    for (int s = 1; s <= B; ++s) {
        // The planes' LDS addresses are kept from one step to the next, in 34
        // registers; the form that has none left for them computes them anew (it
        // spilled nine, which made the loads wait for each other; elsewhere that
        // costs up to 3% of a run).
        int fp = FP;
        if constexpr (B == 3 && BZ == 8 && sizeof(T) == 8 && BC == 0 && RED) asm volatile("" : "+s"(fp));
        if (s > 1) __syncthreads();
        if (in) {
#pragma unroll
            for (int z = s; z < FZ - s; ++z) SM[(z - 1) * fp + tid] = cur[z];
        }
        __syncthreads();
        T below = cur[s - 1];
#pragma unroll
        for (int z = s; z < FZ - s; ++z) {
            const T *P = SM + (z - 1) * fp;
            const T c = cur[z];
            const T s6 = ((P[xm] + P[xp]) + (P[ym] + P[yp])) + (below + cur[z + 1]);
            const T lapn = fma(T(-6), c, s6);
            T nv;
            const T qv = ADJ && s == 2 ? q2[z < (ADJ ? FZ : 1) ? z : 0] : q1[z];
            if constexpr (ADJ) {
                nv = fma(C0, lapn, c);
                nv = fma(-(C1 * qv) * qv, c, nv);
            } else {
                nv = fma(C2, qv, c);
                nv = fma(C0, lapn, nv);
                nv = fma(-(C1 * c) * c, c, nv);
            }
            const int gz = z0 - B + z;
            if (z >= B && z < B + BZ) {
                if constexpr (RED) {
                    double t0 = s0[s - 1], t1 = s1[s - 1];
                    if constexpr (ADJ) {
                        const double du = (double)qv;
                        t0 = fma((double)lapn, du, t0);
                        t1 = fma((double)c, du * du * du, t1);
                    } else {
                        const double d = (double)nv;
                        t0 = fma(d, d, t0);
                        const double dd = d - (double)c;
                        t1 = fma(dd, dd, t1);
                    }
                    s0[s - 1] = gz < nz ? t0 : s0[s - 1];
                    s1[s - 1] = gz < nz ? t1 : s1[s - 1];
                }
                if constexpr (LAM) lv[z >= B && z - B < BZ ? z - B : 0] += c;
            }
            if constexpr (BC == 0) nv = ghost || gz < 0 || gz >= nz ? T(0) : nv;
            below = c;
            cur[z] = nv;
            // four planes' LDS reads in flight
            if ((z - s) % 4 == 3) __builtin_amdgcn_sched_barrier(0);
        }
        void *dst = s < B ? a.mid[s < B ? s - 1 : 0] : a.out;
        if (dst && own) {
#pragma unroll
            for (int z = B; z < B + BZ; ++z)
                if (z0 - B + z < nz)
                    __builtin_nontemporal_store(cur[z], static_cast<T *>(dst) + (int64_t)(z0 - B + z) * sz + col);
        }
    }
    if constexpr (LAM) {
        if (own) {
#pragma unroll
            for (int z = 0; z < BZ; ++z)
                if (z0 + z < nz)
                    __builtin_nontemporal_store(lv[z], static_cast<T *>(a.lam) + (int64_t)(z0 + z) * sz + col);
        }
    }
    if (!own) {
#pragma unroll
        for (int s = 0; s < B; ++s) s0[s] = s1[s] = 0.0;
    }

    if constexpr (RED) {
        // butterfly within the wave, then the waves in order
        double *red = reinterpret_cast<double *>(blk_smem);
        const int lane = tid & 63, wave = tid >> 6, nw = kLanes / 64;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
#pragma unroll
            for (int s = 0; s < B; ++s) {
                s0[s] += __shfl_xor(s0[s], off, 64);
                s1[s] += __shfl_xor(s1[s], off, 64);
            }
        }
        __syncthreads();
        if (lane == 0) {
#pragma unroll
            for (int s = 0; s < B; ++s) {
                red[2 * B * wave + 2 * s] = s0[s];
                red[2 * B * wave + 2 * s + 1] = s1[s];
            }
        }
        __syncthreads();
        if (tid < 2 * B) {
            double x = 0.0;
            for (int w = 0; w < nw; ++w) x += red[2 * B * w + tid];
            a.part[tid / 2][2 * (int64_t)Lb + tid % 2] = x;
        }
    }
}

template <typename T, int B, int BZ>
hipError_t blk_launch_t(int op, int bc, bool reduce, const BlkTile &t, const BlkArgs &a, hipStream_t st) {
    const dim3 grid(t.nblk), block(kLanes);
#define DCP_BLK(BCV, OPV, REDV)                                                                       \
    do {                                                                                              \
        auto fn = block_kernel<T, B, BZ, BCV, OPV, REDV>;                                             \
        hipError_t e_ = hipFuncSetAttribute(reinterpret_cast<const void *>(fn),                       \
                                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)t.lds);  \
        if (e_ != hipSuccess) return e_;                                                              \
        hipLaunchKernelGGL(fn, grid, block, t.lds, st, a);                                            \
    } while (0)
    if (op == SOP_FWD) {
        if (bc == 0) {
            if (reduce) DCP_BLK(0, SOP_FWD, true);
            else DCP_BLK(0, SOP_FWD, false);
        } else {
            if (reduce) DCP_BLK(1, SOP_FWD, true);
            else DCP_BLK(1, SOP_FWD, false);
        }
        return hipGetLastError();
    }
    if constexpr (B == 2) {
        if (op == SOP_ADJ) {
            if (bc == 0) DCP_BLK(0, SOP_ADJ, true);
            else DCP_BLK(1, SOP_ADJ, true);
            return hipGetLastError();
        }
        if (op == SOP_ADJL) {
            if (bc == 0) DCP_BLK(0, SOP_ADJL, true);
            else DCP_BLK(1, SOP_ADJL, true);
            return hipGetLastError();
        }
    }
#undef DCP_BLK
    return hipErrorInvalidValue;
}

}  // namespace

bool blk_plan(int dtype, int B, int64_t nx, int64_t ny, int64_t nz, size_t lds_limit, BlkTile *t) {
    const size_t esz = dtype == 0 ? 8 : 4;
    if (B < 2 || B > 3 || nx <= 0 || ny <= 0 || nz <= 0) return false;
    if (nx > (1 << 24) || ny > (1 << 24) || nx * ny > (int64_t)INT32_MAX || nz > (1 << 24)) return false;
    // The block with the smallest frame that covers the grid with one workgroup
    // per CU.  With a second round the marching forms are faster (us per step,
    // FP64, three steps per pass: 64^3 5.0 marching, 3.8 over blocks; 96^3 6.2
    // and 4.8; 101 x 97 x 103, two rounds, 7.2 and 8.7; 128^3 8.2 and 12.5).
    int64_t best = INT64_MAX;
    bool found = false;
    for (int bz : {4, 8}) {
        const int64_t nbz = (nz + bz - 1) / bz;
        if (nbz > 256) continue;
        for (int64_t nbx = 1; nbx * nbz <= 256 && nbx <= nx; ++nbx) {
            const int64_t bx = (nx + nbx - 1) / nbx, fx = bx + 2 * B;
            int64_t by = kLanes / fx - 2 * B;
            if (by < 1) continue;
            const int64_t nby = (ny + by - 1) / by;
            by = (ny + nby - 1) / nby;
            const int64_t nblk = nbx * nby * nbz, fy = by + 2 * B;
            if (nblk > 256) continue;
            const size_t lds = std::max((size_t)(fx * fy) * (size_t)(bz + 2 * B - 2) * esz,
                                        (size_t)(kLanes / 64) * 2 * B * sizeof(double));
            const int64_t cost = fx * fy * (bz + 2 * B);
            if (lds > lds_limit || cost >= best) continue;
            best = cost;
            found = true;
            t->B = B;
            t->bx = (int)bx;
            t->by = (int)by;
            t->bz = bz;
            t->tiles_x = (int)nbx;
            t->tiles_y = (int)nby;
            t->nblk = (int)nblk;
            t->lds = lds;
        }
    }
    return found;
}

hipError_t launch_blk(int dtype, int op, int bc, bool reduce, const BlkTile &t, const BlkArgs &a, hipStream_t st) {
#define DCP_BLK_T(TT)                                                                                   \
    do {                                                                                                \
        if (t.B == 2 && t.bz == 4) return blk_launch_t<TT, 2, 4>(op, bc, reduce, t, a, st);             \
        if (t.B == 2 && t.bz == 8) return blk_launch_t<TT, 2, 8>(op, bc, reduce, t, a, st);             \
        if (t.B == 3 && t.bz == 4) return blk_launch_t<TT, 3, 4>(op, bc, reduce, t, a, st);             \
        if (t.B == 3 && t.bz == 8) return blk_launch_t<TT, 3, 8>(op, bc, reduce, t, a, st);             \
    } while (0)
    if (dtype == 0) DCP_BLK_T(double);
    else DCP_BLK_T(float);
#undef DCP_BLK_T
    return hipErrorInvalidValue;
}

}  // namespace dcp
