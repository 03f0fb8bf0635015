// dcp_api.cpp -- C ABI of libdcp (declared in include/dcp.h): argument
// checks, workspace layout, tile choice and the host drivers of the time
// loop and of the checkpointed adjoint.  All device work is enqueued on the
// caller's stream; nothing here synchronises or allocates device memory.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <initializer_list>
#include <mutex>
#include <vector>

#include "dcp.h"
#include "dcp_internal.h"

using namespace dcp;

namespace {

constexpr size_t kAlign = 256;
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

struct Geo {
    int64_t nx = 0, ny = 0, nz = 0, n = 0;
    size_t esz = 8;
    size_t bytes() const { return (size_t)n * esz; }
};

int check_geo(int dtype, int64_t nx, int64_t ny, int64_t nz, Geo *g) {
    if (dtype != DCP_F64 && dtype != DCP_F32) return DCP_E_DTYPE;
    if (nx < 0 || ny < 0 || nz < 0) return DCP_E_SHAPE;
    const int64_t ext_lim = (int64_t)1 << 30;
    if (nx > ext_lim || ny > ext_lim || nz > ext_lim) return DCP_E_SHAPE;
    g->esz = dtype == DCP_F64 ? 8 : 4;
    g->nx = nx;
    g->ny = ny;
    g->nz = nz;
    g->n = 0;
    if (nx && ny && nz) {
        const int64_t lim = ((int64_t)1 << 60) / (int64_t)g->esz;
        if (nx > lim / ny) return DCP_E_SHAPE;
        const int64_t nxy = nx * ny;
        if (nxy > lim / nz) return DCP_E_SHAPE;
        g->n = nxy * nz;
    }
    return DCP_OK;
}

int check_coeffs(const dcp_coeffs *c) {
    if (!c) return DCP_E_NULL;
    const double v[5] = {c->alpha, c->beta, c->gamma, c->h, c->dt};
    for (double x : v)
        if (!std::isfinite(x)) return DCP_E_ARG;
    if (!(c->h > 0.0)) return DCP_E_ARG;
    return DCP_OK;
}

bool aligned16(const void *p) { return ((uintptr_t)p & 15u) == 0; }

bool overlaps(const void *a, size_t na, const void *b, size_t nb) {
    if (!a || !b || na == 0 || nb == 0) return false;
    const uintptr_t a0 = (uintptr_t)a, b0 = (uintptr_t)b;
    return a0 < b0 + nb && b0 < a0 + na;
}

// ------------------------------------------------------------- tile choice
int env_int(const char *name, int def) {
    const char *s = tuning_env(name);
    if (!s || !*s) return def;
    return std::atoi(s);
}

Tile make_tile(const Geo &g, int vec, int shape, int zc) {
    Tile t{};
    const Shape s = shape_at(shape);
    t.vec = vec;
    t.bxw = s.bxw;
    t.by = s.by;
    t.ry = s.ry;
    t.zc = zc;
    const int64_t tx = (g.nx + (int64_t)64 * s.bxw * vec - 1) / ((int64_t)64 * s.bxw * vec);
    const int64_t ty = (g.ny + (int64_t)s.by * s.ry - 1) / ((int64_t)s.by * s.ry);
    const int64_t tz = (g.nz + zc - 1) / zc;
    const int64_t nb = tx * ty * tz;
    t.tiles_x = (int)tx;
    t.tiles_y = (int)ty;
    t.tiles_z = (int)tz;
    t.nblk = nb > INT32_MAX / 1024 ? -1 : (int)nb;
    return t;
}

// Most workgroups of a step whose sums are reduced (its pairs of sums are
// stored), and of one without.
constexpr int kSumBlocks = 8192, kPlainBlocks = 32768;

// What a tile's step does: a forward step without sums or with them, or an adjoint
// step.
enum StepUse { kPlainStep, kSumStep, kAdjointStep };

// Tile of the one-step kernels.  A wave covers 64 vectors of one row; a lane
// holds two rows (shape 1: 8 rows per workgroup, four waves per SIMD) or four
// (shape 0: 16 rows, two waves per SIMD, fewer rows read twice), and marches up
// runs of zc planes, two of which it shares with the next run.  512 workgroups
// of shape 0 run at once, or 1024 of shape 1.  The rule goes by how many of shape
// 0 with runs of 8 planes the grid gives; times in us per step (with norms, unless
// "plain"), the other choice first:
//   * under 410, four fifths of a round: shape 1, in runs of 8 planes, fewer
//     where that leaves under 1200 workgroups (FP32: 900), so that every CU has
//     work: FP64 64^3 12.2 / 4.9, 96^3 14.1 / 7.8, 128^3 20.4 / 16.1;
//   * up to 512, one round nearly or just full: shape 0, whose runs share less:
//     FP32 512 x 512 x 64 40.4 / 38.5, 384 x 706 x 37 34.3 / 31.0; plain steps,
//     which pay less for a run, runs of 2 of shape 1 (FP64 160^3 27.1 / 25.0);
//   * between 512 and 896, and 1024 and 1152, where a last round would be nearly
//     empty: shape 1, whose rounds are finer (FP64 192^3 46.8 / 42.2); just under
//     1024 shape 0 again (FP32 908 x 168 x 175 69.0 / 66.2; plain, runs of 4 of
//     shape 1);
//   * more: shape 0 in runs of 8 (FP64 512^3 584 / 567, FP32 298 / 285), of 4
//     where the step is plain (FP64 360 x 388 x 475 311 / 284).  With norms, runs of 7
//     where those end closer to the grid's last plane (FP64 640 x 500 x 300 454 / 442,
//     FP32 223 / 218; 190 grids 0.3% in the mean, none over 3% slower).  Single grids
//     prefer 4 to 16 planes by up to 12%, in no order found;
//   * rows just longer than a wave's, which leave over two fifths of their waves
//     idle, run long in shape 0: FP64 136 x 748 x 425 plain 263.7 in runs of 4, 256.2
//     in runs of 16.
// Narrow rows, which fill at most three quarters of one wave (48 vectors), have
// few points to a plane's halo loads: shape 1 keeps four waves per SIMD waiting
// on them.  FP64 24 x 360 x 1157 130.7 / 114.7, plain 129.5 in runs of 4 / 102.9;
// FP32 128 x 720 x 542 130.0 / 116.9.  With sums, rows of at most half a wave
// run 16 planes where that leaves two rounds (FP64 24 x 720 x 2893 559 / 525).
// FP32 rows of at most 48 points take single elements (31 x 360 x 896: 90.9 with
// vectors, 84.4; plain 73.1 / 64.4; at 62 points 51.8 / 50.9).
// Adjoint steps hold more registers, the more with the running sum of their inputs or
// where they recompute their state (which leaves four rows per lane one wave per
// SIMD): they take shape 1 as grids under 410 do, and shape 0 where that would be too
// many workgroups.  FP64 992 x 72 x 235 160 / 142, FP32 231 x 515 x 273 with the sum 237 /
// 181, 200 steps of the reverse sweep of 256^3 FP64 33.0 / 31.1 ms; only one full round is
// the better in shape 0 without the sum (FP32 256^3 40.0 / 41.6).  All of them take one
// tile: the parameter sums are the same, bit for bit, with the running sum and without.
// Single elements on FP32 rows of at most 64 points that are not whole vectors (45 x
// 400 x 666 80 / 74, with the sum 149 / 144; 63 x 400 x 476 60 / 55 and 135 / 111).
// Past kSumBlocks or kPlainBlocks workgroups the runs grow, up to 64 planes.
// DCP_TILE_SHAPE / DCP_TILE_ZC override the choice in tuning runs (with
// DCP_TUNING=1).
Tile pick_tile(int dtype, const Geo &g, bool vec_ok, StepUse use) {
    const bool sums = use != kPlainStep;
    const int wide = dtype == DCP_F64 ? 2 : 4, most = sums ? kSumBlocks : kPlainBlocks;
    const int forced = env_int("DCP_TILE_SHAPE", -1);
    int shape = forced >= 0 && forced < num_shapes() ? forced : -1;
    const bool adjoint = use == kAdjointStep, ragged = g.nx % wide != 0;
    // (vectors on ragged rows are compiled for the two shapes chosen here)
    const bool one = !vec_ok || (ragged && shape > 1) ||
                     (dtype == DCP_F32 && (adjoint ? ragged && g.nx <= 64 : g.nx <= 48));
    const int vec = one ? 1 : wide;
    auto blocks = [&](int sh, int z) {
        const int nb = make_tile(g, vec, sh, z).nblk;
        return nb < 0 ? INT32_MAX : nb;
    };
    auto at_least = [&](int sh, int z, int lo, int nb) {  // runs of z planes, halved down to lo while under nb workgroups
        while (z > lo && blocks(sh, z) < nb) z /= 2;
        return z;
    };
    int zc = env_int("DCP_TILE_ZC", 0);
    if (zc <= 0) {
        const int n8 = blocks(0, 8);
        const int64_t span = (g.nx + 64 * vec - 1) / (64 * vec) * 64 * vec;  // points the row's waves could hold
        auto pick = [&](int sh, int z) {
            if (shape < 0) shape = sh;
            zc = z;
        };
        auto few = [&] {
            const int z = at_least(1, 8, 2, dtype == DCP_F64 ? 1200 : 900);
            pick(1, z == 2 && blocks(1, 2) < 512 ? 1 : z);
        };
        const bool narrow = g.nx <= 48 * vec;
        if (one) {
            if (sums) pick(0, at_least(0, adjoint ? 4 : 8, 1, 700));
            else pick(1, at_least(1, 4, 1, 700));
        } else if (adjoint && blocks(1, 8) > most) {
            pick(0, 8);
        } else if (adjoint || n8 < 410) {
            few();
        } else if (n8 <= 512) {
            if (sums) pick(0, 8);
            else if (narrow) few();
            else pick(1, 2);
        } else if (narrow) {
            const int z = sums && g.nx <= 32 * vec && blocks(1, 16) >= 2048 ? 16 : 8;
            if (dtype == DCP_F64 && blocks(1, z) > most) pick(0, at_least(0, 64, 8, 2048));
            else pick(1, z);
        } else if (n8 < 896) {
            few();
        } else if (n8 < 1024) {
            if (sums) pick(0, 8);
            else pick(1, 4);
        } else if (n8 < 1152) {
            pick(1, 8);
        } else if (10 * g.nx < 6 * span) {
            pick(0, at_least(0, 64, 8, 2048));
        } else {
            const bool seven = (g.nz + 6) / 7 * 7 < (g.nz + 7) / 8 * 8 && blocks(0, 7) <= most;
            pick(0, !sums ? 4 : seven ? 7 : 8);
        }
        while (zc < 64 && blocks(shape, zc) > most) zc *= 2;
        if (forced != shape && blocks(shape, zc) > most) shape = 0;
    }
    if (shape < 0) shape = 1;
    if (g.nz > 0 && zc > g.nz) zc = (int)g.nz;
    if (zc < 1) zc = 1;
    return make_tile(g, vec, shape, zc);
}

// Largest workgroup count of a step with sums over both vector widths
// (workspace sizing must not depend on pointer alignment).
int max_blocks(int dtype, const Geo &g, StepUse use) {
    if (g.n == 0) return 0;
    const Tile a = pick_tile(dtype, g, true, use), b = pick_tile(dtype, g, false, use);
    if (a.nblk < 0 || b.nblk < 0) return -1;
    return std::max(a.nblk, b.nblk);
}

// ---------------------------------------------------------- workspace layout
struct StepWs {
    size_t temps = 0;     // offset of 3 temporaries (unfused)
    size_t partials = 0;  // offset of partial sums
    size_t total = 0;
};

int layout_step(int dtype, int impl, const Geo &g, bool norms, StepWs *w) {
    size_t off = 0;
    if (impl == DCP_UNFUSED && g.n > 0) {
        w->temps = off;
        off += 3 * align_up(g.bytes());
    }
    if (norms && g.n > 0) {
        const int nb = impl == DCP_UNFUSED ? ew_norm_blocks(g.n) : max_blocks(dtype, g, kSumStep);
        if (nb < 0) return DCP_E_SHAPE;
        w->partials = off;
        off += align_up((size_t)nb * 2 * sizeof(double));
    }
    w->total = off;
    return DCP_OK;
}

// Steps whose workgroups' pairs of sums a workspace holds at once, at most T:
// 16 MiB of them (512^3: 128 steps) and a pass's three at least.  Longer runs
// reduce a batch when it is full, one launch in a batch's time, and the
// workspace does not grow with the steps.
int32_t sum_steps(int32_t T, int nblk) {
    const size_t fit = ((size_t)16 << 20) / ((size_t)nblk * 2 * sizeof(double));
    return (int32_t)std::min<size_t>((size_t)T, fit < 3 ? 3 : fit);
}

struct RunWs {
    size_t field = 0;     // ping-pong field
    size_t temps = 0;     // unfused temporaries
    size_t partials = 0;  // [sum_steps][nblk][2]
    int nblk = 0;
    size_t total = 0;
};

// LDS of one workgroup on gfx950, the most a two-step pass may plan for.
constexpr size_t kLdsMax = 160 * 1024;

// Plan of a B-step pass (dcp_tbk.hip): for three steps the ring form (768
// lanes) where a tile fits it, else 1024 lanes; for two steps the reverse.  DCP_TBK_CFG="wc,ty,lanes" restricts the
// planner to segments of wc chunks (a value covering the row: whole rows),
// slabs of ty rows and 768, 1024 or 512 lanes; 0 leaves a choice to the
// planner.  DCP_TBK_SBLK sets the slabs per block of the tile order.
// Tuning overrides only: every choice computes the same states bit for bit
// (the norms' summation order follows the tiles).
bool tbk_for(int dtype, const Geo &g, int B, bool vok, size_t lds_limit, TbkTile *t) {
    int wc = 0, ty = 0, lanes = 0;
    if (const char *e = tuning_env("DCP_TBK_CFG")) {
        int a = 0, b = 0, c = 0;
        if (std::sscanf(e, "%d,%d,%d", &a, &b, &c) == 3) {
            wc = a > 0 ? a : 0;
            ty = b > 0 ? b : 0;
            lanes = c == 512 || c == 768 || c == 1024 ? c : 0;
        }
    }
    // measured at 1024x1024x512 FP64: the ring form is the faster for three
    // steps per pass (22.4 against 24.7 ms for T = 24), the plain form for
    // two (30.7 against 34.4 ms)
    const int first = B == 3 ? 768 : 1024, second = B == 3 ? 1024 : 768;
    bool ok = false;
    if (lanes) ok = tbk_plan(dtype, B, g.nx, g.ny, g.nz, vok, lds_limit, lanes, wc, ty, t);
    else ok = tbk_plan(dtype, B, g.nx, g.ny, g.nz, vok, lds_limit, first, wc, ty, t) ||
              tbk_plan(dtype, B, g.nx, g.ny, g.nz, vok, lds_limit, second, wc, ty, t);
    if (!ok) return false;
    if (const char *e = tuning_env("DCP_TBK_SBLK")) {
        const int h = std::atoi(e);
        if (h > 0) t->sblk = h < t->nslab ? h : t->nslab;
    }
    return true;
}

// Plan of a B-step pass over blocks (dcp_block.hip), the first choice on small
// grids; off while a tuning override forces one of the marching forms.
bool blk_for(int dtype, const Geo &g, int B, size_t lds_limit, BlkTile *t) {
    for (const char *name : {"DCP_TB_CFG", "DCP_TBK_CFG"})
        if (const char *e = tuning_env(name); e && *e) return false;
    return blk_plan(dtype, B, g.nx, g.ny, g.nz, lds_limit, t);
}

int layout_run(int dtype, int impl, const Geo &g, int32_t T, int32_t tblock, bool norms, RunWs *w) {
    size_t off = 0;
    if (g.n == 0 || T == 0) {
        w->total = 0;
        return DCP_OK;
    }
    w->field = off;
    off += align_up(g.bytes());
    if (impl == DCP_UNFUSED) {
        w->temps = off;
        off += 3 * align_up(g.bytes());
    }
    if (norms) {
        int nb = impl == DCP_UNFUSED ? ew_norm_blocks(g.n) : max_blocks(dtype, g, kSumStep);
        if (nb < 0) return DCP_E_SHAPE;
        TbTile tb;
        if (impl == DCP_FUSED && tblock >= 2 && tb_plan(dtype, g.nx, g.ny, g.nz, true, kLdsMax, &tb) &&
            tb.nblk > nb)
            nb = tb.nblk;
        for (int B = 2; impl == DCP_FUSED && B <= tblock && B <= 3; ++B) {
            TbkTile tk;
            if (tbk_for(dtype, g, B, true, kLdsMax, &tk) && tk.nblk > nb) nb = tk.nblk;
            BlkTile bk;
            if (blk_for(dtype, g, B, kLdsMax, &bk) && bk.nblk > nb) nb = bk.nblk;
        }
        w->nblk = nb;
        w->partials = off;
        off += align_up((size_t)sum_steps(T, nb) * nb * 2 * sizeof(double));
    }
    w->total = off;
    return DCP_OK;
}

struct AdjWs {
    size_t lam = 0;       // 2 fields
    size_t seg = 0;       // k-1 fields
    size_t partials = 0;  // [sum_steps][nblk][2]
    size_t sums = 0;      // [T][2]
    size_t lsum = 0;      // 1 field: running sum of the adjoint inputs (when wanted there)
    size_t dot = 0;       // [ew_norm_blocks][2] + 2: partials of <sum, f>
    int nblk = 0;
    size_t total = 0;
};

// lsum_field: reserve the running-sum field (dL/dgamma without a grad_f buffer).
int layout_adj(int dtype, const Geo &g, int32_t T, int32_t k, int32_t tblock, bool lsum_field, AdjWs *w) {
    size_t off = 0;
    if (T == 0) {
        w->total = 0;
        return DCP_OK;
    }
    if (g.n > 0) {
        int nb = max_blocks(dtype, g, kAdjointStep);
        if (nb < 0) return DCP_E_SHAPE;
        TbTile tb;
        if (tblock >= 2 && tb_plan(dtype, g.nx, g.ny, g.nz, true, kLdsMax, &tb) && tb.nblk > nb) nb = tb.nblk;
        BlkTile bk;
        if (tblock >= 2 && blk_for(dtype, g, 2, kLdsMax, &bk) && bk.nblk > nb) nb = bk.nblk;
        w->nblk = nb;
        w->lam = off;
        off += 2 * align_up(g.bytes());
        w->seg = off;
        const int32_t kk = k < T ? k : T;
        off += (size_t)(kk - 1) * align_up(g.bytes());
        w->partials = off;
        off += align_up((size_t)sum_steps(T, nb) * nb * 2 * sizeof(double));
        if (lsum_field) {
            w->lsum = off;
            off += align_up(g.bytes());
        }
        w->dot = off;
        off += align_up(((size_t)ew_norm_blocks(g.n) * 2 + 2) * sizeof(double));
    }
    w->sums = off;
    off += align_up((size_t)T * 2 * sizeof(double));
    w->total = off;
    return DCP_OK;
}

int check_ws(const void *ws, size_t ws_bytes, size_t need) {
    if (need == 0) return DCP_OK;
    if (ws_bytes < need) return DCP_E_WORKSPACE;
    if (!ws) return DCP_E_NULL;
    return DCP_OK;
}

char *at(void *base, size_t off) { return static_cast<char *>(base) + off; }

int hip_status(hipError_t e) { return e == hipSuccess ? DCP_OK : DCP_E_HIP; }

#define DCP_TRY(expr)                            \
    do {                                         \
        hipError_t e_ = (expr);                  \
        if (e_ != hipSuccess) return DCP_E_HIP;  \
    } while (0)

// The per-workgroup pairs of sums of a sweep's steps, in the workspace's room for
// sum_steps of them: step s in slot s mod that many, the steps held consecutive.
// A batch is reduced when the next steps do not fit beside it, and at the end, in
// a fixed order, one launch for each run of steps that share a workgroup count.
class StepSums {
  public:
    StepSums(double *partials, int stride, int32_t T, int nblk, double *out0, double *out1, int mode, hipStream_t st)
        : p_(partials), stride_(stride), cap_(stride > 0 ? sum_steps(T, stride) : 0), out0_(out0), out1_(out1),
          mode_(mode), st_(st) {
        if (p_) nblk_.assign((size_t)T, nblk);
    }
    // Takes steps lo .. hi - 1, next to those held.
    hipError_t take(int32_t lo, int32_t hi) {
        if (!p_) return hipSuccess;
        if (std::max(hi, hi_) - std::min(lo, lo_) > cap_ || lo_ == hi_) {
            if (hipError_t e = reduce()) return e;
            lo_ = lo;
            hi_ = hi;
        } else {
            lo_ = std::min(lo, lo_);
            hi_ = std::max(hi, hi_);
        }
        return hipSuccess;
    }
    double *of(int32_t s) const { return p_ ? p_ + (size_t)(s % cap_) * stride_ * 2 : nullptr; }
    void set(int32_t lo, int32_t hi, int nblk) {
        if (p_) std::fill(nblk_.begin() + lo, nblk_.begin() + hi, nblk);
    }
    hipError_t reduce() {
        for (int32_t s0 = lo_; s0 < hi_;) {
            int32_t s1 = s0 + 1;
            while (s1 < hi_ && s1 % cap_ != 0 && nblk_[s1] == nblk_[s0]) ++s1;
            double *o0 = out0_ ? out0_ + (size_t)s0 * (mode_ == 2 ? 2 : 1) : nullptr;
            if (hipError_t e = launch_finalize(of(s0), nblk_[s0], stride_, s1 - s0, o0, out1_ ? out1_ + s0 : nullptr,
                                               mode_, st_))
                return e;
            s0 = s1;
        }
        lo_ = hi_ = 0;
        return hipSuccess;
    }

  private:
    double *p_;
    int stride_;
    int32_t cap_, lo_ = 0, hi_ = 0;
    double *out0_, *out1_;
    int mode_;
    hipStream_t st_;
    std::vector<int> nblk_;  // workgroups behind each step's pairs
};

StencilArgs fwd_args(const Geo &g, const dcp_coeffs &c, const Tile &t, const void *u, const void *f,
                     void *out, double *partials) {
    StencilArgs a{};
    a.s = u;
    a.q = f;
    a.out = out;
    a.partials = partials;
    a.nx = g.nx;
    a.ny = g.ny;
    a.nz = g.nz;
    a.c0 = c.dt * c.alpha / (c.h * c.h);
    a.c1 = c.dt * c.beta;
    a.c2 = c.dt * c.gamma;
    a.tiles_x = t.tiles_x;
    a.tiles_y = t.tiles_y;
    a.zc = t.zc;
    a.nblk = t.nblk;
    return a;
}

// One fused step u -> out (partials may be null).
hipError_t fused_step(int dtype, int bc, const Geo &g, const dcp_coeffs &c, const Tile &t, const void *u,
                      const void *f, void *out, double *partials, hipStream_t st) {
    const StencilArgs a = fwd_args(g, c, t, u, f, out, partials);
    return launch_stencil(dtype, SOP_FWD, bc, partials != nullptr, t, a, st);
}

// One unfused step (the single-operator statements), temporaries in tmp[3].
hipError_t unfused_step(int dtype, int bc, const Geo &g, const dcp_coeffs &c, const Tile &t, bool vec_ok,
                        const void *u, const void *f, void *out, void *const tmp[3], double *partials,
                        hipStream_t st) {
    void *A = tmp[0], *B = tmp[1], *C = tmp[2];
    StencilArgs a{};
    a.s = u;
    a.q = nullptr;
    a.out = A;
    a.partials = nullptr;
    a.nx = g.nx;
    a.ny = g.ny;
    a.nz = g.nz;
    a.c0 = c.h * c.h;
    a.tiles_x = t.tiles_x;
    a.tiles_y = t.tiles_y;
    a.zc = t.zc;
    a.nblk = t.nblk;
    hipError_t e;
    if ((e = launch_stencil(dtype, SOP_LAP, bc, false, t, a, st)) != hipSuccess) return e;  // lap = Lap7(u)  -> A
    if ((e = launch_ew(dtype, EW_POW3, u, nullptr, B, 0.0, g.n, vec_ok, st))) return e;     // u3 = (u*u)*u  -> B
    if ((e = launch_ew(dtype, EW_SCALE, A, nullptr, C, c.alpha, g.n, vec_ok, st))) return e;  // t1 = alpha*lap -> C
    if ((e = launch_ew(dtype, EW_SCALE, B, nullptr, A, c.beta, g.n, vec_ok, st))) return e;   // t2 = beta*u3  -> A
    if ((e = launch_ew(dtype, EW_SUB, C, A, B, 0.0, g.n, vec_ok, st))) return e;              // t3 = t1 - t2  -> B
    if ((e = launch_ew(dtype, EW_SCALE, f, nullptr, C, c.gamma, g.n, vec_ok, st))) return e;  // t4 = gamma*f  -> C
    if ((e = launch_ew(dtype, EW_ADD, B, C, A, 0.0, g.n, vec_ok, st))) return e;              // t5 = t3 + t4  -> A
    if ((e = launch_ew(dtype, EW_SCALE, A, nullptr, B, c.dt, g.n, vec_ok, st))) return e;     // t6 = dt*t5    -> B
    if ((e = launch_ew(dtype, EW_ADD, u, B, out, 0.0, g.n, vec_ok, st))) return e;            // u' = u + t6
    if (partials) return launch_ew_norms(dtype, out, u, partials, g.n, vec_ok, st);
    return hipSuccess;
}

// A two-step pass u_t -> u_{t+2} (mid receives u_{t+1} when not null).
hipError_t tb_fwd_pass(int dtype, int bc, const Geo &g, const dcp_coeffs &c, const TbTile &tb, const void *u,
                       const void *f, void *out, void *mid, double *part1, double *part2, hipStream_t st) {
    TbArgs ta{};
    ta.u = u;
    ta.f = f;
    ta.out = out;
    ta.mid = mid;
    ta.part1 = part1;
    ta.part2 = part2;
    ta.nx = g.nx;
    ta.ny = g.ny;
    ta.nz = g.nz;
    ta.c0 = c.dt * c.alpha / (c.h * c.h);
    ta.c1 = c.dt * c.beta;
    ta.c2 = c.dt * c.gamma;
    ta.nslab = tb.nslab;
    ta.zc = tb.zc;
    return launch_tb2(dtype, SOP_FWD, bc, part1 != nullptr, tb, ta, st);
}

// LDS one workgroup may use on the current device (gfx950's 160 KiB when no
// device can be asked, for plans made on a host without one).
size_t device_lds() {
    int dev = 0, lds = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess || lds <= 0)
        return kLdsMax;
    return (size_t)lds;
}

// Plans a two-step pass when asked for and supported by the grid and device.
bool plan_tb(int dtype, const Geo &g, int32_t tblock, bool vok, TbTile *tb) {
    if (tblock < 2) return false;
    return tb_plan(dtype, g.nx, g.ny, g.nz, vok, device_lds(), tb);
}

// Plans a B-step pass (B = 2, 3) when the grid and the device allow it.
bool plan_tbk(int dtype, const Geo &g, int B, bool vok, TbkTile *t) {
    return tbk_for(dtype, g, B, vok, device_lds(), t);
}

// Smallest ragged grid that takes passes of several steps.  The line is the marching
// forms': at 64^3 points their three-step pass takes as long as three single steps
// (17 us against 18), at 101 x 97 x 103 23 us against 26, at 257 x 263 x 255 98
// against 290.  Blocks do not depend on it, and a grid below it would take 0.60 to
// 0.81 of the time over them (48 steps of 63^3 FP64 237 us, 162 over blocks), but the
// plan of a small ragged grid is one step per pass to its callers.
constexpr int64_t kRaggedMin = (int64_t)1 << 18;

// The passes of a fused dcp_run: three steps where tblock >= 3 and the
// B-step kernel applies; two steps over whole rows where the two-step kernel
// applies, else over x-segments; one step otherwise and for the remainders.
// Small grids take two and three steps over blocks.
// stride: partial-sum slots per step of the run's workspace (norms only).
struct PassPlan {
    bool use_tb = false, use_k2 = false, use_k3 = false;
    bool use_b2 = false, use_b3 = false;  // over blocks, before the others
    TbTile tb{};
    TbkTile k2{}, k3{};
    BlkTile b2{}, b3{};
    // steps in the pass starting at step s of T: three where possible, but
    // four steps left go as two passes of two (cheaper than three and one)
    int32_t len_at(int32_t s, int32_t T) const {
        const bool two = use_tb || use_k2 || use_b2;
        if ((use_k3 || use_b3) && s + 3 <= T && !(two && T - s == 4)) return 3;
        if (two && s + 2 <= T) return 2;
        return 1;
    }
};

PassPlan plan_passes(int dtype, int impl, const Geo &g, int32_t T, int32_t tblock, bool vok, bool norms,
                     int stride) {
    PassPlan pp;
    if (impl != DCP_FUSED) return pp;
    // ragged rows (not whole vectors): over x-segments, on grids that are worth it
    const bool ragged = g.nx % (dtype == DCP_F64 ? 2 : 4) != 0;
    if (ragged && g.n < kRaggedMin) return pp;
    const size_t lds = device_lds();
    pp.use_b2 = T >= 2 && tblock >= 2 && vok && blk_for(dtype, g, 2, lds, &pp.b2) && (!norms || pp.b2.nblk <= stride);
    pp.use_b3 = T >= 3 && tblock >= 3 && vok && blk_for(dtype, g, 3, lds, &pp.b3) && (!norms || pp.b3.nblk <= stride);
    pp.use_tb = T >= 2 && !ragged && plan_tb(dtype, g, tblock, vok, &pp.tb) && (!norms || pp.tb.nblk <= stride);
    pp.use_k2 = !pp.use_tb && T >= 2 && tblock >= 2 && plan_tbk(dtype, g, 2, vok, &pp.k2) &&
                (!norms || pp.k2.nblk <= stride);
    pp.use_k3 = T >= 3 && tblock >= 3 && plan_tbk(dtype, g, 3, vok, &pp.k3) && (!norms || pp.k3.nblk <= stride);
    return pp;
}

// A B-step pass u_t -> u_{t+B}; mid[s-1] receives u_{t+s} when not null;
// part (when not null) holds the B steps' partial-sum arrays.
hipError_t tbk_fwd_pass(int dtype, int bc, const Geo &g, const dcp_coeffs &c, const TbkTile &tk, const void *u,
                        const void *f, void *out, void *const mid[2], double *const part[3], hipStream_t st) {
    TbkArgs a{};
    a.u = u;
    a.f = f;
    a.out = out;
    for (int i = 0; i < 2; ++i) a.mid[i] = mid ? mid[i] : nullptr;
    for (int i = 0; i < 3; ++i) a.part[i] = part ? part[i] : nullptr;
    a.nx = g.nx;
    a.ny = g.ny;
    a.nz = g.nz;
    a.c0 = c.dt * c.alpha / (c.h * c.h);
    a.c1 = c.dt * c.beta;
    a.c2 = c.dt * c.gamma;
    a.ty = tk.ty;
    a.nslab = tk.nslab;
    a.nseg = tk.nseg;
    a.zc = tk.zc;
    a.wc = tk.wc;
    a.halo = tk.halo;
    a.chf = tk.chf;
    a.sblk = tk.sblk;
    a.shift = tk.shift;
    return launch_tbk(dtype, bc, part != nullptr, tk, a, st);
}

// A pass of bk.B steps over blocks u_t -> u_{t+B}; mid and part as above.
hipError_t blk_fwd_pass(int dtype, int bc, const Geo &g, const dcp_coeffs &c, const BlkTile &bk, const void *u,
                        const void *f, void *out, void *const mid[2], double *const part[3], hipStream_t st) {
    BlkArgs a{};
    a.u = u;
    a.q[0] = f;
    a.out = out;
    for (int i = 0; i < 2; ++i) a.mid[i] = mid ? mid[i] : nullptr;
    for (int i = 0; i < 3; ++i) a.part[i] = part ? part[i] : nullptr;
    a.nx = g.nx;
    a.ny = g.ny;
    a.nz = g.nz;
    a.c0 = c.dt * c.alpha / (c.h * c.h);
    a.c1 = c.dt * c.beta;
    a.c2 = c.dt * c.gamma;
    a.bx = bk.bx;
    a.by = bk.by;
    a.tiles_x = bk.tiles_x;
    a.tiles_y = bk.tiles_y;
    return launch_blk(dtype, SOP_FWD, bc, part != nullptr, bk, a, st);
}

// Two adjoint steps per pass, on grids whose rows fit a whole-row tile: over
// blocks where the grid is small, else over whole rows; nblk = 0 where there
// are none (or `stride` partial slots are too few).
struct PairPlan {
    TbTile tb{};
    BlkTile bk{};
    bool blocks = false;
    int nblk = 0;
};

// Whether pairs over whole rows pay on rows that are not whole vectors.  A plane of a
// tile's run takes as long on short rows, which leave most of its 1024 lanes idle, where
// single steps take less.  The rule prices a pair by its planes in sequence and the
// chunks of a plane's frame, two single steps by the grid's rows and their points, us,
// each with a launch; fitted to 478 gradients on 239 such grids, with the running sum and
// without.  Four steps, us, single and in pairs: FP32 31 x 700 x 1612 1090 / 2510, 161 x
// 700 x 310 369 / 595, 255 x 400 x 98 116 / 100, 818 x 157 x 103 with the sum 317 / 171;
// FP64 31 x 700 x 1612 1370 / 2220, 255 x 400 x 98 223 / 135.  Against single elements
// the choice gains 2.21x in the mean and 0.95x at the least, always pairs 2.12x and
// 0.45x, never 1.69x and 0.95x.  With the running sum pairs pay a little sooner (FP32 74 x
// 147 x 266, four steps: 123 us, single 155): one choice for both keeps the parameter
// sums the same.  Rows of whole vectors take pairs throughout.
bool pair_pays(int dtype, const Geo &g, const TbTile &tb) {
    const bool f64 = dtype == DCP_F64;
    const double frame = (double)(tb.ty + 4) * (double)((g.nx + tb.vec - 1) / tb.vec), launch = f64 ? 6.5 : 7.8;
    const double planes = (double)((tb.nblk + 255) / 256) * (double)(tb.zc + 4), rows = 1e-3 * (double)(g.ny * g.nz);
    const double pair = launch + planes * (f64 ? 1.61 + 0.000375 * frame : 0.73 + 0.000717 * frame);
    const double step = launch + rows * (f64 ? 0.328 + 0.0046 * (double)g.nx : 0.067 + 0.0016 * (double)g.nx);
    return pair <= 2.0 * step;
}

PairPlan plan_pair(int dtype, const Geo &g, int32_t tblock, bool vok, int stride) {
    PairPlan p;
    if (!plan_tb(dtype, g, tblock, vok, &p.tb)) return p;  // pairs where rows fit a whole-row tile
    p.blocks = blk_for(dtype, g, 2, device_lds(), &p.bk) && p.bk.nblk <= stride;
    const bool ragged = g.nx % (dtype == DCP_F64 ? 2 : 4) != 0;
    if (p.blocks) p.nblk = p.bk.nblk;
    else if (p.tb.nblk <= stride && (!ragged || pair_pays(dtype, g, p.tb))) p.nblk = p.tb.nblk;
    return p;
}

hipError_t adj_pair(int dtype, int op, int bc, const PairPlan &p, const TbArgs &ta, hipStream_t st) {
    if (!p.blocks) return launch_tb2(dtype, op, bc, true, p.tb, ta, st);
    BlkArgs a{};
    a.u = ta.u;
    a.q[0] = ta.f;
    a.q[1] = ta.g2;
    a.out = ta.out;
    a.lam = ta.lam;
    a.part[0] = ta.part1;
    a.part[1] = ta.part2;
    a.nx = ta.nx;
    a.ny = ta.ny;
    a.nz = ta.nz;
    a.c0 = ta.c0;
    a.c1 = ta.c1;
    a.bx = p.bk.bx;
    a.by = p.bk.by;
    a.tiles_x = p.bk.tiles_x;
    a.tiles_y = p.bk.tiles_y;
    a.lam_first = ta.lam_first;
    return launch_blk(dtype, op, bc, true, p.bk, a, st);
}

// One forward pass of len (1, 2 or 3) steps without norms, u -> out, in the
// kernel `pp` plans for that length; mid[i] (when not null) receives the
// state after i+1 steps of a multi-step pass.
hipError_t fwd_pass(int dtype, int bc, const Geo &g, const dcp_coeffs &c, const Tile &t, const PassPlan &pp,
                    int len, const void *u, const void *f, void *out, void *mid0, void *mid1, hipStream_t st) {
    if ((len == 3 && pp.use_b3) || (len == 2 && pp.use_b2)) {
        void *mid[2] = {mid0, len == 3 ? mid1 : nullptr};
        return blk_fwd_pass(dtype, bc, g, c, len == 3 ? pp.b3 : pp.b2, u, f, out, mid, nullptr, st);
    }
    if (len == 3 || (len == 2 && !pp.use_tb)) {
        void *mid[2] = {mid0, len == 3 ? mid1 : nullptr};
        return tbk_fwd_pass(dtype, bc, g, c, len == 3 ? pp.k3 : pp.k2, u, f, out, mid, nullptr, st);
    }
    if (len == 2) return tb_fwd_pass(dtype, bc, g, c, pp.tb, u, f, out, mid0, nullptr, nullptr, st);
    return fused_step(dtype, bc, g, c, t, u, f, out, nullptr, st);
}

// 16-byte lanes of the stencil kernels: rows of at least one vector, pointers
// aligned to their elements (global vectors need no more).
bool vec_ok_for(int dtype, const Geo &g, std::initializer_list<const void *> ptrs) {
    if (g.nx < (dtype == DCP_F64 ? 2 : 4)) return false;
    for (const void *p : ptrs)
        if ((uintptr_t)p % g.esz != 0) return false;
    return true;
}

// The element-wise kernels run over the flat field: 16-byte aligned pointers.
bool ew_ok(std::initializer_list<const void *> ptrs) {
    for (const void *p : ptrs)
        if (p && !aligned16(p)) return false;
    return true;
}

int step_common(int impl, int dtype, const void *u, const void *f, void *u_out, int64_t nx, int64_t ny,
                int64_t nz, const dcp_coeffs *coeffs, int bc, double *norms2, void *ws, size_t ws_bytes,
                void *stream) {
    Geo g;
    int rc = check_geo(dtype, nx, ny, nz, &g);
    if (rc) return rc;
    if (bc != DCP_DIRICHLET0 && bc != DCP_PERIODIC) return DCP_E_BC;
    if ((rc = check_coeffs(coeffs))) return rc;
    if (g.n > 0 && (!u || !f || !u_out)) return DCP_E_NULL;
    StepWs w;
    if ((rc = layout_step(dtype, impl, g, norms2 != nullptr, &w))) return rc;
    if ((rc = check_ws(ws, ws_bytes, w.total))) return rc;
    const size_t fb = g.bytes();
    if (overlaps(u_out, fb, u, fb) || overlaps(u_out, fb, f, fb)) return DCP_E_ALIAS;
    if (overlaps(ws, w.total, u, fb) || overlaps(ws, w.total, f, fb) || overlaps(ws, w.total, u_out, fb))
        return DCP_E_ALIAS;
    if (norms2 && (overlaps(norms2, 16, u, fb) || overlaps(norms2, 16, f, fb) ||
                   overlaps(norms2, 16, u_out, fb) || overlaps(norms2, 16, ws, w.total)))
        return DCP_E_ALIAS;

    hipStream_t st = static_cast<hipStream_t>(stream);
    if (g.n == 0) return norms2 ? hip_status(launch_zero(norms2, 2, st)) : DCP_OK;

    double *partials = norms2 ? reinterpret_cast<double *>(at(ws, w.partials)) : nullptr;
    if (impl == DCP_FUSED) {
        const Tile t = pick_tile(dtype, g, vec_ok_for(dtype, g, {u, f, u_out}), norms2 ? kSumStep : kPlainStep);
        DCP_TRY(fused_step(dtype, bc, g, *coeffs, t, u, f, u_out, partials, st));
        if (norms2) DCP_TRY(launch_finalize(partials, t.nblk, t.nblk, 1, norms2, nullptr, 0, st));
    } else {
        void *tmp[3] = {at(ws, w.temps), at(ws, w.temps + align_up(fb)), at(ws, w.temps + 2 * align_up(fb))};
        const bool vok = vec_ok_for(dtype, g, {u, f, u_out, tmp[0], tmp[1], tmp[2]});
        const Tile t = pick_tile(dtype, g, vok, kSumStep);
        const bool eok = ew_ok({u, f, u_out, tmp[0], tmp[1], tmp[2]});
        DCP_TRY(unfused_step(dtype, bc, g, *coeffs, t, eok, u, f, u_out, tmp, partials, st));
        if (norms2) {
            const int nb = ew_norm_blocks(g.n);
            DCP_TRY(launch_finalize(partials, nb, nb, 1, norms2, nullptr, 0, st));
        }
    }
    return DCP_OK;
}

int32_t num_slots(int32_t T, int32_t k) { return T <= 0 ? 0 : (T + k - 1) / k; }

// ------------------------------------------------ binomial checkpointing
// Workspace of the two revolve calls (kept by the caller between them):
// the saved u_0, nslots snapshot slots, the work state, an advance scratch
// field, two adjoint fields, optionally the running sum of the adjoint
// inputs, and the reduction scratch of the adjoint.
struct RevWs {
    size_t origin = 0, slots = 0, work = 0, scratch = 0, lam = 0, lsum = 0;
    size_t partials = 0, sums = 0, dot = 0;
    int nblk = 0;
    size_t total = 0;
};

int layout_rev(int dtype, const Geo &g, int32_t T, int32_t nslots, bool lsum_field, RevWs *w) {
    size_t off = 0;
    if (T == 0 || g.n == 0) {
        w->total = 0;
        return DCP_OK;
    }
    const size_t fb = align_up(g.bytes());
    int nb = max_blocks(dtype, g, kAdjointStep);
    if (nb < 0) return DCP_E_SHAPE;
    BlkTile bk;
    if (blk_for(dtype, g, 2, kLdsMax, &bk) && bk.nblk > nb) nb = bk.nblk;
    w->nblk = nb;
    w->origin = off;
    off += fb;
    w->slots = off;
    off += (size_t)nslots * fb;
    w->work = off;
    off += fb;
    w->scratch = off;
    off += fb;
    w->lam = off;
    off += 2 * fb;
    if (lsum_field) {
        w->lsum = off;
        off += fb;
    }
    w->partials = off;
    off += align_up((size_t)sum_steps(T, nb) * nb * 2 * sizeof(double));
    w->sums = off;
    off += align_up((size_t)T * 2 * sizeof(double));
    w->dot = off;
    off += align_up(((size_t)ew_norm_blocks(g.n) * 2 + 2) * sizeof(double));
    w->total = off;
    return DCP_OK;
}

struct RevBufs {
    void *ws;
    const RevWs *w;
    int32_t nslots;
    size_t fb;
    void *buf(int32_t id) const {
        if (id == kRvOrigin) return at(ws, w->origin);
        if (id < nslots) return at(ws, w->slots + (size_t)id * fb);
        return at(ws, w->work);
    }
};

// n fused steps from `from` into `to` (n >= 1; both distinct from the
// scratch field), in the passes of `pp` (up to three steps each where the
// grid allows it), alternating between `to` and the scratch so the last pass
// lands in `to`.
int rev_advance(int dtype, int bc, const Geo &g, const dcp_coeffs &c, const Tile &t, const PassPlan &pp,
                const void *f, const void *from, void *to, void *scratch, int64_t n, hipStream_t st) {
    std::vector<int> lens;
    for (int64_t left = n; left > 0;) {
        const int k = pp.len_at(0, (int32_t)std::min<int64_t>(left, INT32_MAX));
        lens.push_back(k);
        left -= k;
    }
    const void *cur = from;
    const size_t L = lens.size();
    for (size_t i = 0; i < L; ++i) {
        void *out = ((L - 1 - i) % 2 == 0) ? to : scratch;
        if (fwd_pass(dtype, bc, g, c, t, pp, lens[i], cur, f, out, nullptr, nullptr, st) != hipSuccess)
            return DCP_E_HIP;
        cur = out;
    }
    return DCP_OK;
}

}  // namespace

extern "C" {

const char *dcp_status_string(int status) {
    switch (status) {
        case DCP_OK: return "ok";
        case DCP_E_NULL: return "a required pointer is NULL";
        case DCP_E_SHAPE: return "invalid grid shape (negative extent or size overflow)";
        case DCP_E_DTYPE: return "invalid dtype (expected DCP_F64 or DCP_F32)";
        case DCP_E_BC: return "invalid boundary (expected DCP_DIRICHLET0 or DCP_PERIODIC)";
        case DCP_E_ARG: return "invalid argument (T, ckpt_every, tblock, h, impl, op or a non-finite coefficient)";
        case DCP_E_WORKSPACE: return "workspace too small";
        case DCP_E_ALIAS: return "an output overlaps an input";
        case DCP_E_SCRATCH:
            return "the grid needs more than the 1 MiB device scratch of the allocation-free entry point";
        case DCP_E_HIP: return "HIP launch or copy failed";
        default: return "unknown status";
    }
}

int32_t dcp_max_tblock(int dtype) { return (dtype == DCP_F64 || dtype == DCP_F32) ? 3 : 1; }

int dcp_workspace_bytes(int op, int dtype, int impl, int64_t nx, int64_t ny, int64_t nz, int32_t T,
                        int32_t ckpt_every, int32_t tblock, int norms, size_t *bytes) {
    if (!bytes) return DCP_E_NULL;
    Geo g;
    int rc = check_geo(dtype, nx, ny, nz, &g);
    if (rc) return rc;
    switch (op) {
        case DCP_OP_STEP_FUSED:
        case DCP_OP_STEP_UNFUSED: {
            StepWs w;
            if ((rc = layout_step(dtype, op == DCP_OP_STEP_FUSED ? DCP_FUSED : DCP_UNFUSED, g, norms != 0, &w)))
                return rc;
            *bytes = w.total;
            return DCP_OK;
        }
        case DCP_OP_RUN: {
            if (impl != DCP_FUSED && impl != DCP_UNFUSED) return DCP_E_ARG;
            if (T < 0 || tblock < 1 || tblock > dcp_max_tblock(dtype)) return DCP_E_ARG;
            RunWs w;
            if ((rc = layout_run(dtype, impl, g, T, tblock, norms != 0, &w))) return rc;
            *bytes = w.total;
            return DCP_OK;
        }
        case DCP_OP_ADJOINT: {
            if (T < 0 || ckpt_every < 1) return DCP_E_ARG;
            if (tblock < 1 || tblock > dcp_max_tblock(dtype)) return DCP_E_ARG;
            AdjWs w;
            if ((rc = layout_adj(dtype, g, T, ckpt_every, tblock, norms != 0, &w))) return rc;
            *bytes = w.total;
            return DCP_OK;
        }
        default: return DCP_E_ARG;
    }
}

int dcp_step_fused(int dtype, const void *u, const void *f, void *u_out, int64_t nx, int64_t ny, int64_t nz,
                   const dcp_coeffs *coeffs, int bc, double *norms2, void *ws, size_t ws_bytes, void *stream) {
    return step_common(DCP_FUSED, dtype, u, f, u_out, nx, ny, nz, coeffs, bc, norms2, ws, ws_bytes, stream);
}

// ------------------------------------------------ allocation-free fused step
// Scratch of dcp_step_fused_noalloc: the norms' per-workgroup partial sums.
// Every GPU holds its own copy (with the code object) until the process
// ends.  In host code `scratch` names a host-side stand-in, never the device
// memory: kernels and copies get the address hipGetSymbolAddress returns for
// the current device, fetched once per device.
static __device__ __align__(256) double scratch[DCP_NOALLOC_SCRATCH_BYTES / sizeof(double)];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};

int scratch_of_current_device(void **out) {
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return DCP_E_HIP;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) return DCP_E_HIP;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return DCP_OK;
}

}  // namespace

int dcp_step_fused_noalloc(int dtype, const void *u, const void *f, void *u_out, int64_t nx, int64_t ny,
                           int64_t nz, const dcp_coeffs *coeffs, int bc, double *norms2, void *stream) {
    // argument errors first (the same checks as dcp_step_fused), then the size
    Geo g;
    int rc = check_geo(dtype, nx, ny, nz, &g);
    if (rc) return rc;
    if (bc != DCP_DIRICHLET0 && bc != DCP_PERIODIC) return DCP_E_BC;
    if ((rc = check_coeffs(coeffs))) return rc;
    if (g.n > 0 && (!u || !f || !u_out)) return DCP_E_NULL;
    StepWs w;
    if ((rc = layout_step(dtype, DCP_FUSED, g, norms2 != nullptr, &w))) return rc;
    if (w.total > DCP_NOALLOC_SCRATCH_BYTES) return DCP_E_SCRATCH;
    const size_t fb = g.bytes();
    if (overlaps(u_out, fb, u, fb) || overlaps(u_out, fb, f, fb)) return DCP_E_ALIAS;
    if (norms2 && (overlaps(norms2, 16, u, fb) || overlaps(norms2, 16, f, fb) || overlaps(norms2, 16, u_out, fb)))
        return DCP_E_ALIAS;
    void *ws = nullptr;
    if (w.total > 0 && (rc = scratch_of_current_device(&ws))) return rc;
    return step_common(DCP_FUSED, dtype, u, f, u_out, nx, ny, nz, coeffs, bc, norms2, ws,
                       w.total > 0 ? (size_t)DCP_NOALLOC_SCRATCH_BYTES : 0, stream);
}

int dcp_step_unfused(int dtype, const void *u, const void *f, void *u_out, int64_t nx, int64_t ny, int64_t nz,
                     const dcp_coeffs *coeffs, int bc, double *norms2, void *ws, size_t ws_bytes, void *stream) {
    return step_common(DCP_UNFUSED, dtype, u, f, u_out, nx, ny, nz, coeffs, bc, norms2, ws, ws_bytes, stream);
}

int dcp_run(int dtype, int impl, void *u, const void *f, int64_t nx, int64_t ny, int64_t nz,
            const dcp_coeffs *coeffs, int bc, int32_t T, int32_t tblock, double *energy, double *resid,
            void *ckpt, int32_t ckpt_every, void *ws, size_t ws_bytes, void *stream) {
    Geo g;
    int rc = check_geo(dtype, nx, ny, nz, &g);
    if (rc) return rc;
    if (bc != DCP_DIRICHLET0 && bc != DCP_PERIODIC) return DCP_E_BC;
    if ((rc = check_coeffs(coeffs))) return rc;
    if (impl != DCP_FUSED && impl != DCP_UNFUSED) return DCP_E_ARG;
    if (T < 0 || tblock < 1 || tblock > dcp_max_tblock(dtype)) return DCP_E_ARG;
    if (tblock > 1 && impl != DCP_FUSED) return DCP_E_ARG;
    if (ckpt && ckpt_every < 1) return DCP_E_ARG;
    if (g.n > 0 && (!u || !f)) return DCP_E_NULL;
    const bool norms = energy || resid;
    RunWs w;
    if ((rc = layout_run(dtype, impl, g, T, tblock, norms, &w))) return rc;
    if ((rc = check_ws(ws, ws_bytes, w.total))) return rc;
    const size_t fb = g.bytes();
    const int32_t nslots = ckpt ? num_slots(T, ckpt_every) : 0;
    const size_t cb = (size_t)nslots * fb;
    const size_t nb = (size_t)(T > 0 ? T : 0) * sizeof(double);
    if (overlaps(u, fb, f, fb)) return DCP_E_ALIAS;
    if (overlaps(ws, w.total, u, fb) || overlaps(ws, w.total, f, fb)) return DCP_E_ALIAS;
    if (overlaps(ckpt, cb, u, fb) || overlaps(ckpt, cb, f, fb) || overlaps(ckpt, cb, ws, w.total))
        return DCP_E_ALIAS;
    for (const double *o : {energy, resid})
        if (o && (overlaps(o, nb, u, fb) || overlaps(o, nb, f, fb) || overlaps(o, nb, ws, w.total) ||
                  overlaps(o, nb, ckpt, cb)))
            return DCP_E_ALIAS;
    if (energy && resid && overlaps(energy, nb, resid, nb)) return DCP_E_ALIAS;

    hipStream_t st = static_cast<hipStream_t>(stream);
    if (T == 0) return DCP_OK;
    if (g.n == 0) {
        if (energy) DCP_TRY(launch_zero(energy, T, st));
        if (resid) DCP_TRY(launch_zero(resid, T, st));
        return DCP_OK;
    }

    void *buf = at(ws, w.field);
    void *tmp[3] = {nullptr, nullptr, nullptr};
    if (impl == DCP_UNFUSED)
        for (int i = 0; i < 3; ++i) tmp[i] = at(ws, w.temps + i * align_up(fb));
    auto slot = [&](int32_t c) { return static_cast<void *>(static_cast<char *>(ckpt) + (size_t)c * fb); };
    const bool vok = vec_ok_for(dtype, g, {u, f, buf, tmp[0], tmp[1], tmp[2], ckpt});
    bool eok = ew_ok({u, f, buf, tmp[0], tmp[1], tmp[2]});  // of every state and temporary
    for (int32_t c = 0; c < nslots; ++c) eok = eok && aligned16(slot(c));
    const Tile t = pick_tile(dtype, g, vok, kSumStep);
    const int nblk_one = impl == DCP_UNFUSED ? ew_norm_blocks(g.n) : t.nblk;
    const int stride = w.nblk;  // partial slots per step (>= every kernel's workgroup count)
    double *partials = norms ? reinterpret_cast<double *>(at(ws, w.partials)) : nullptr;

    // passes of several steps where the grid allows them and the device has
    // the LDS: three steps (tblock 3), two steps over whole rows (tblock >= 2,
    // rows that fit the LDS) or over x-segments (longer rows)
    const PassPlan pp = plan_passes(dtype, impl, g, T, tblock, vok, norms, stride);
    const bool use_tb = pp.use_tb;
    const TbTile &tb = pp.tb;
    const TbkTile &tk2 = pp.k2, &tk3 = pp.k3;

    StepSums step_sums(partials, stride, T, nblk_one, energy, resid, 1, st);

    auto is_ckpt = [&](int32_t t) { return nslots > 0 && t % ckpt_every == 0 && t / ckpt_every < nslots; };
    if (nslots > 0) DCP_TRY(launch_ew(dtype, EW_COPY, u, nullptr, slot(0), 0.0, g.n, ew_ok({u, slot(0)}), st));
    const void *cur = u;
    for (int32_t s = 0; s < T;) {
        const int32_t len = pp.len_at(s, T);
        const int32_t se = s + len;
        void *nxt = is_ckpt(se) ? slot(se / ckpt_every) : ((cur == u) ? buf : u);
        DCP_TRY(step_sums.take(s, se));
        double *p = step_sums.of(s);
        const bool blocks = (len == 3 && pp.use_b3) || (len == 2 && pp.use_b2);
        if (len == 3 || (len == 2 && (blocks || !use_tb))) {
            // checkpoints at the middle steps are stored by the pass itself
            const TbkTile &tk = len == 3 ? tk3 : tk2;
            const BlkTile &bk = len == 3 ? pp.b3 : pp.b2;
            void *mid[2] = {is_ckpt(s + 1) ? slot((s + 1) / ckpt_every) : nullptr,
                            len == 3 && is_ckpt(s + 2) ? slot((s + 2) / ckpt_every) : nullptr};
            double *part[3] = {p, step_sums.of(s + 1), len == 3 ? step_sums.of(s + 2) : nullptr};
            if (blocks) DCP_TRY(blk_fwd_pass(dtype, bc, g, *coeffs, bk, cur, f, nxt, mid, p ? part : nullptr, st));
            else DCP_TRY(tbk_fwd_pass(dtype, bc, g, *coeffs, tk, cur, f, nxt, mid, p ? part : nullptr, st));
            step_sums.set(s, se, blocks ? bk.nblk : tk.nblk);
        } else if (len == 2) {
            // a checkpoint at the middle step is stored by the pass itself
            void *mid = is_ckpt(s + 1) ? slot((s + 1) / ckpt_every) : nullptr;
            DCP_TRY(tb_fwd_pass(dtype, bc, g, *coeffs, tb, cur, f, nxt, mid, p, step_sums.of(s + 1), st));
            step_sums.set(s, se, tb.nblk);
        } else if (impl == DCP_FUSED) {
            DCP_TRY(fused_step(dtype, bc, g, *coeffs, t, cur, f, nxt, p, st));
        } else {
            DCP_TRY(unfused_step(dtype, bc, g, *coeffs, t, eok, cur, f, nxt, tmp, p, st));
        }
        cur = nxt;
        s = se;
    }
    if (cur != u) DCP_TRY(launch_ew(dtype, EW_COPY, cur, nullptr, u, 0.0, g.n, ew_ok({cur, u}), st));
    DCP_TRY(step_sums.reduce());
    return DCP_OK;
}

int dcp_run_plan(int dtype, int impl, int64_t nx, int64_t ny, int64_t nz, int32_t T, int32_t tblock, int norms,
                 dcp_run_info *info) {
    if (!info) return DCP_E_NULL;
    Geo g;
    int rc = check_geo(dtype, nx, ny, nz, &g);
    if (rc) return rc;
    if (impl != DCP_FUSED && impl != DCP_UNFUSED) return DCP_E_ARG;
    if (T < 0 || tblock < 1 || tblock > dcp_max_tblock(dtype)) return DCP_E_ARG;
    if (tblock > 1 && impl != DCP_FUSED) return DCP_E_ARG;
    RunWs w;
    if ((rc = layout_run(dtype, impl, g, T, tblock, norms != 0, &w))) return rc;
    std::memset(info, 0, sizeof(*info));
    if (T == 0 || g.n == 0) return DCP_OK;
    const int wide = dtype == DCP_F64 ? 2 : 4;
    const PassPlan pp = plan_passes(dtype, impl, g, T, tblock, g.nx >= wide, norms != 0, w.nblk);
    int32_t most = 0;
    for (int32_t s = 0; s < T;) {
        const int32_t len = pp.len_at(s, T);
        ++info->passes[len - 1];
        most = len > most ? len : most;
        s += len;
    }
    info->steps_per_pass = most;
    if (most >= 2 && (most == 3 ? pp.use_b3 : pp.use_b2)) {
        const BlkTile &bk = most == 3 ? pp.b3 : pp.b2;
        info->segmented = bk.bx < g.nx ? 1 : 0;
        info->tile_rows = bk.by;
        info->lanes = kBlkLanes;
    } else if (most >= 2) {
        const bool k = most == 3 || !pp.use_tb;
        const TbkTile &tk = most == 3 ? pp.k3 : pp.k2;
        info->segmented = k && tk.seg ? 1 : 0;
        info->tile_rows = k ? tk.ty : pp.tb.ty;
        info->lanes = k ? tk.nt : 1024;
    }
    return DCP_OK;
}

int dcp_adjoint_run(int dtype, const void *ckpt, int32_t ckpt_every, const void *f, const void *lam_T, int64_t nx,
                    int64_t ny, int64_t nz, const dcp_coeffs *coeffs, int bc, int32_t T, int32_t tblock,
                    void *grad_u0, double *grad_ab, void *grad_f, double *grad_gamma, void *ws, size_t ws_bytes,
                    void *stream) {
    Geo g;
    int rc = check_geo(dtype, nx, ny, nz, &g);
    if (rc) return rc;
    if (bc != DCP_DIRICHLET0 && bc != DCP_PERIODIC) return DCP_E_BC;
    if ((rc = check_coeffs(coeffs))) return rc;
    if (T < 0 || ckpt_every < 1 || tblock < 1 || tblock > dcp_max_tblock(dtype)) return DCP_E_ARG;
    if (!grad_ab) return DCP_E_NULL;
    if (g.n > 0 && (!f || !lam_T || !grad_u0 || (T > 0 && !ckpt))) return DCP_E_NULL;
    const bool lsum_field = grad_gamma != nullptr && grad_f == nullptr && g.n > 0;
    AdjWs w;
    if ((rc = layout_adj(dtype, g, T, ckpt_every, tblock, lsum_field, &w))) return rc;
    if ((rc = check_ws(ws, ws_bytes, w.total))) return rc;
    const size_t fb = g.bytes();
    const int32_t nslots = num_slots(T, ckpt_every);
    const size_t cb = (size_t)nslots * fb;
    if (overlaps(grad_u0, fb, ckpt, cb) || overlaps(grad_u0, fb, f, fb) || overlaps(grad_u0, fb, lam_T, fb) ||
        overlaps(grad_u0, fb, ws, w.total))
        return DCP_E_ALIAS;
    if (overlaps(ws, w.total, ckpt, cb) || overlaps(ws, w.total, f, fb) || overlaps(ws, w.total, lam_T, fb))
        return DCP_E_ALIAS;
    if (overlaps(grad_ab, 16, grad_u0, fb) || overlaps(grad_ab, 16, ws, w.total) || overlaps(grad_ab, 16, ckpt, cb))
        return DCP_E_ALIAS;
    if (grad_f && (overlaps(grad_f, fb, ckpt, cb) || overlaps(grad_f, fb, f, fb) || overlaps(grad_f, fb, lam_T, fb) ||
                   overlaps(grad_f, fb, grad_u0, fb) || overlaps(grad_f, fb, ws, w.total) ||
                   overlaps(grad_f, fb, grad_ab, 16)))
        return DCP_E_ALIAS;
    if (grad_gamma && (overlaps(grad_gamma, 8, grad_ab, 16) || overlaps(grad_gamma, 8, grad_u0, fb) ||
                       overlaps(grad_gamma, 8, grad_f, grad_f ? fb : 0) || overlaps(grad_gamma, 8, ws, w.total) ||
                       overlaps(grad_gamma, 8, ckpt, cb)))
        return DCP_E_ALIAS;

    hipStream_t st = static_cast<hipStream_t>(stream);
    if (T == 0 || g.n == 0) {
        if (g.n > 0)
            DCP_TRY(launch_ew(dtype, EW_COPY, lam_T, nullptr, grad_u0, 0.0, g.n,
                              ew_ok({lam_T, grad_u0}), st));
        if (grad_f && g.n > 0)
            DCP_TRY(launch_ew(dtype, EW_ZERO, nullptr, nullptr, grad_f, 0.0, g.n, ew_ok({grad_f}), st));
        DCP_TRY(launch_zero(grad_ab, 2, st));
        if (grad_gamma) DCP_TRY(launch_zero(grad_gamma, 1, st));
        return DCP_OK;
    }
    // running sum of the adjoint inputs lambda_T .. lambda_1 (for dL/df and dL/dgamma)
    void *lsum = grad_f ? grad_f : (lsum_field ? static_cast<void *>(at(ws, w.lsum)) : nullptr);

    void *lam[2] = {at(ws, w.lam), at(ws, w.lam + align_up(fb))};
    const int32_t kk = ckpt_every < T ? ckpt_every : T;
    auto seg = [&](int32_t j) { return static_cast<void *>(at(ws, w.seg + (size_t)j * align_up(fb))); };
    auto slot = [&](int32_t c) { return static_cast<const void *>(static_cast<const char *>(ckpt) + (size_t)c * fb); };
    const bool vok = vec_ok_for(dtype, g, {f, lam_T, grad_u0, lam[0], lam[1], lsum, ckpt, seg(0)});
    const Tile t = pick_tile(dtype, g, vok, kAdjointStep);
    const Tile tf = pick_tile(dtype, g, vok, kPlainStep);  // recomputation
    double *partials = reinterpret_cast<double *>(at(ws, w.partials));
    double *sums = reinterpret_cast<double *>(at(ws, w.sums));
    const int stride = w.nblk;
    const dcp_coeffs &c = *coeffs;
    const PairPlan ap = plan_pair(dtype, g, tblock, vok, stride);
    const PassPlan fpp = plan_passes(dtype, DCP_FUSED, g, T, tblock, vok, false, 0);  // recomputation

    StencilArgs aa{};
    aa.nx = g.nx;
    aa.ny = g.ny;
    aa.nz = g.nz;
    aa.c0 = c.dt * c.alpha / (c.h * c.h);
    aa.c1 = 3.0 * c.dt * c.beta;
    aa.tiles_x = t.tiles_x;
    aa.tiles_y = t.tiles_y;
    aa.zc = t.zc;
    aa.nblk = t.nblk;
    TbArgs ta{};
    ta.nx = g.nx;
    ta.ny = g.ny;
    ta.nz = g.nz;
    ta.c0 = aa.c0;
    ta.c1 = aa.c1;
    ta.nslab = ap.tb.nslab;
    ta.zc = ap.tb.zc;

    // Adjoint steps are taken in pairs (2m+1, 2m) by global parity, whatever
    // the checkpoint interval: a pair whose lower step lies in the previous
    // segment waits for that segment (its upper state is a checkpoint slot).
    // Every step's parameter sums therefore come from the same kernel with the
    // same tiling for any k, and the gradient does not depend on k bit for bit.
    StepSums step_sums(partials, stride, T, t.nblk, sums, nullptr, 2, st);
    const int adj_op = lsum ? SOP_ADJL : SOP_ADJ;
    aa.lam = lsum;
    ta.lam = lsum;
    int lam_first = 1;
    const void *lcur = lam_T;
    int32_t s = T - 1;  // next adjoint step to take
    for (int32_t cs = nslots - 1; cs >= 0; --cs) {
        const int32_t t0 = cs * ckpt_every;
        const int32_t t1 = (t0 + ckpt_every < T) ? t0 + ckpt_every : T;
        // recompute the states u_{t0+1} .. u_{t1-1} of this segment (u_{t0+j}
        // into seg(j-1)), up to three steps per pass, every state stored
        const void *prev = slot(cs);
        for (int32_t j = 1; j < t1 - t0;) {
            const int32_t left = t1 - t0 - j;
            const int len = fpp.len_at(0, left);
            DCP_TRY(fwd_pass(dtype, bc, g, c, tf, fpp, len, prev, f, seg(j + len - 2),
                             len >= 2 ? seg(j - 1) : nullptr, len == 3 ? seg(j) : nullptr, st));
            prev = seg(j + len - 2);
            j += len;
        }
        // u_t for t in [t0, t1], the upper end being the next slot
        auto state = [&](int32_t tt) -> const void * {
            if (tt % ckpt_every == 0) return slot(tt / ckpt_every);
            return seg(tt - t0 - 1);
        };
        while (s >= t0) {
            const bool pair = ap.nblk && (s & 1) && s >= 1;
            if (pair && s - 1 < t0) break;  // the lower step lives in the previous segment
            const int32_t se = pair ? s - 1 : s;
            DCP_TRY(step_sums.take(se, s + 1));
            void *out = (se == 0) ? grad_u0 : (lcur == lam[0] ? lam[1] : lam[0]);
            if (pair) {
                ta.u = lcur;
                ta.f = state(s);
                ta.g2 = state(s - 1);
                ta.out = out;
                ta.mid = nullptr;
                ta.part1 = step_sums.of(s);
                ta.part2 = step_sums.of(s - 1);
                ta.lam_first = lam_first;
                DCP_TRY(adj_pair(dtype, adj_op, bc, ap, ta, st));
                step_sums.set(s - 1, s + 1, ap.nblk);
            } else {
                aa.s = lcur;
                aa.q = state(s);
                aa.out = out;
                aa.partials = step_sums.of(s);
                aa.lam_first = lam_first;
                DCP_TRY(launch_stencil(dtype, adj_op, bc, true, t, aa, st));
            }
            lam_first = 0;
            lcur = out;
            s = se - 1;
        }
    }
    // per-step sums in a fixed order, then over the steps in a fixed order
    DCP_TRY(step_sums.reduce());
    DCP_TRY(launch_grad_finalize(sums, T, c.dt / (c.h * c.h), -c.dt, grad_ab, st));
    if (lsum) {
        // dL/dgamma = dt * <sum, f> (fixed-order double reduction), then
        // dL/df = gamma * dt * sum in place
        if (grad_gamma) {
            double *dp = reinterpret_cast<double *>(at(ws, w.dot));
            const int nb = ew_norm_blocks(g.n);
            double *pair = dp + 2 * (size_t)nb;
            DCP_TRY(launch_ew_dot(dtype, lsum, f, dp, g.n, ew_ok({lsum, f}), st));
            DCP_TRY(launch_finalize(dp, nb, nb, 1, pair, nullptr, 0, st));
            DCP_TRY(launch_scalar_scale(pair, c.dt, grad_gamma, st));
        }
        if (grad_f)
            DCP_TRY(launch_ew(dtype, EW_SCALE, grad_f, nullptr, grad_f, c.gamma * c.dt, g.n,
                              ew_ok({grad_f}), st));
    }
    return DCP_OK;
}

int dcp_revolve_workspace_bytes(int dtype, int64_t nx, int64_t ny, int64_t nz, int32_t T, int32_t nslots,
                                int lsum_field, size_t *bytes) {
    if (!bytes) return DCP_E_NULL;
    Geo g;
    int rc = check_geo(dtype, nx, ny, nz, &g);
    if (rc) return rc;
    if (T < 0 || nslots < 0) return DCP_E_ARG;
    RevWs w;
    if ((rc = layout_rev(dtype, g, T, nslots, lsum_field != 0, &w))) return rc;
    *bytes = w.total;
    return DCP_OK;
}

int dcp_revolve_forward(int dtype, void *u, const void *f, int64_t nx, int64_t ny, int64_t nz,
                        const dcp_coeffs *coeffs, int bc, int32_t T, int32_t nslots, int32_t tblock, void *ws,
                        size_t ws_bytes, void *stream) {
    Geo g;
    int rc = check_geo(dtype, nx, ny, nz, &g);
    if (rc) return rc;
    if (bc != DCP_DIRICHLET0 && bc != DCP_PERIODIC) return DCP_E_BC;
    if ((rc = check_coeffs(coeffs))) return rc;
    if (T < 0 || nslots < 0 || tblock < 1 || tblock > dcp_max_tblock(dtype)) return DCP_E_ARG;
    if (g.n > 0 && (!u || !f)) return DCP_E_NULL;
    RevWs w;
    if ((rc = layout_rev(dtype, g, T, nslots, false, &w))) return rc;
    // the running-sum field, if any, sits after the fields used here
    if ((rc = check_ws(ws, ws_bytes, w.total))) return rc;
    const size_t fb = g.bytes();
    if (overlaps(u, fb, f, fb) || overlaps(ws, ws_bytes, u, fb) || overlaps(ws, ws_bytes, f, fb)) return DCP_E_ALIAS;
    if (T == 0 || g.n == 0) return DCP_OK;
    std::vector<RvOp> ops;
    if (!revolve_schedule(T, nslots, &ops, nullptr)) return DCP_E_ARG;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const RevBufs B{ws, &w, nslots, align_up(fb)};
    void *scratch = at(ws, w.scratch);
    const bool vok = vec_ok_for(dtype, g, {u, f, ws});
    const Tile tf = pick_tile(dtype, g, vok, kPlainStep);
    const PassPlan pp = plan_passes(dtype, DCP_FUSED, g, T, tblock, vok, false, 0);
    const dcp_coeffs &c = *coeffs;
    DCP_TRY(launch_ew(dtype, EW_COPY, u, nullptr, B.buf(kRvOrigin), 0.0, g.n, ew_ok({u, B.buf(kRvOrigin)}), st));
    // the schedule's opening chain of advances, u_0 -> ... -> u_{T-1}, stores
    // the snapshots the reverse sweep starts from
    int32_t last = kRvOrigin;
    for (const RvOp &op : ops) {
        if (op.kind != kRvAdvance) break;
        if ((rc = rev_advance(dtype, bc, g, c, tf, pp, f, B.buf(op.src), B.buf(op.dst), scratch, op.t1 - op.t0,
                              st)))
            return rc;
        last = op.dst;
    }
    DCP_TRY(fused_step(dtype, bc, g, c, tf, B.buf(last), f, u, nullptr, st));  // u_T
    return DCP_OK;
}

int dcp_revolve_adjoint(int dtype, const void *f, const void *lam_T, int64_t nx, int64_t ny, int64_t nz,
                        const dcp_coeffs *coeffs, int bc, int32_t T, int32_t nslots, int32_t tblock,
                        void *grad_u0, double *grad_ab, void *grad_f, double *grad_gamma, void *ws,
                        size_t ws_bytes, void *stream) {
    Geo g;
    int rc = check_geo(dtype, nx, ny, nz, &g);
    if (rc) return rc;
    if (bc != DCP_DIRICHLET0 && bc != DCP_PERIODIC) return DCP_E_BC;
    if ((rc = check_coeffs(coeffs))) return rc;
    if (T < 0 || nslots < 0 || tblock < 1 || tblock > dcp_max_tblock(dtype)) return DCP_E_ARG;
    if (!grad_ab) return DCP_E_NULL;
    if (g.n > 0 && (!f || !lam_T || !grad_u0)) return DCP_E_NULL;
    const bool lsum_field = grad_gamma != nullptr && grad_f == nullptr && g.n > 0;
    RevWs w;
    if ((rc = layout_rev(dtype, g, T, nslots, lsum_field, &w))) return rc;
    if ((rc = check_ws(ws, ws_bytes, w.total))) return rc;
    const size_t fb = g.bytes();
    const size_t wsz = w.total;
    for (const void *p : {f, lam_T})
        if (overlaps(grad_u0, fb, p, fb) || overlaps(ws, wsz, p, fb) || (grad_f && overlaps(grad_f, fb, p, fb)))
            return DCP_E_ALIAS;
    if (overlaps(grad_u0, fb, ws, wsz) || overlaps(grad_ab, 16, ws, wsz) || overlaps(grad_ab, 16, grad_u0, fb))
        return DCP_E_ALIAS;
    if (grad_f && (overlaps(grad_f, fb, ws, wsz) || overlaps(grad_f, fb, grad_u0, fb) ||
                   overlaps(grad_f, fb, grad_ab, 16)))
        return DCP_E_ALIAS;
    if (grad_gamma && (overlaps(grad_gamma, 8, grad_ab, 16) || overlaps(grad_gamma, 8, grad_u0, fb) ||
                       overlaps(grad_gamma, 8, grad_f, grad_f ? fb : 0) || overlaps(grad_gamma, 8, ws, wsz)))
        return DCP_E_ALIAS;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (T == 0 || g.n == 0) {
        if (g.n > 0)
            DCP_TRY(launch_ew(dtype, EW_COPY, lam_T, nullptr, grad_u0, 0.0, g.n,
                              ew_ok({lam_T, grad_u0}), st));
        if (grad_f && g.n > 0)
            DCP_TRY(launch_ew(dtype, EW_ZERO, nullptr, nullptr, grad_f, 0.0, g.n, ew_ok({grad_f}), st));
        DCP_TRY(launch_zero(grad_ab, 2, st));
        if (grad_gamma) DCP_TRY(launch_zero(grad_gamma, 1, st));
        return DCP_OK;
    }
    std::vector<RvOp> ops;
    if (!revolve_schedule(T, nslots, &ops, nullptr)) return DCP_E_ARG;
    const RevBufs B{ws, &w, nslots, align_up(fb)};
    void *scratch = at(ws, w.scratch);
    void *lam[2] = {at(ws, w.lam), at(ws, w.lam + align_up(fb))};
    void *lsum = grad_f ? grad_f : (lsum_field ? static_cast<void *>(at(ws, w.lsum)) : nullptr);
    const bool vok = vec_ok_for(dtype, g, {f, lam_T, grad_u0, grad_f, ws});
    const Tile t = pick_tile(dtype, g, vok, kAdjointStep);
    const Tile tf = pick_tile(dtype, g, vok, kPlainStep);  // recomputation
    const PassPlan pp = plan_passes(dtype, DCP_FUSED, g, T, tblock, vok, false, 0);
    const dcp_coeffs &c = *coeffs;
    double *partials = reinterpret_cast<double *>(at(ws, w.partials));
    double *sums = reinterpret_cast<double *>(at(ws, w.sums));
    const int stride = w.nblk;
    StencilArgs aa{};
    aa.nx = g.nx;
    aa.ny = g.ny;
    aa.nz = g.nz;
    aa.c0 = c.dt * c.alpha / (c.h * c.h);
    aa.c1 = 3.0 * c.dt * c.beta;
    aa.tiles_x = t.tiles_x;
    aa.tiles_y = t.tiles_y;
    aa.zc = t.zc;
    aa.nblk = t.nblk;
    aa.lam = lsum;
    aa.c1f = c.dt * c.beta;  // the forward step's coefficients, for the fused recomputation
    aa.c2f = c.dt * c.gamma;
    // two adjoint steps per pass where both states are at hand (tblock >= 2)
    const PairPlan ap = plan_pair(dtype, g, tblock, vok, stride);
    TbArgs ta{};
    ta.nx = g.nx;
    ta.ny = g.ny;
    ta.nz = g.nz;
    ta.c0 = aa.c0;
    ta.c1 = aa.c1;
    ta.nslab = ap.tb.nslab;
    ta.zc = ap.tb.zc;
    ta.lam = lsum;
    StepSums step_sums(partials, stride, T, t.nblk, sums, nullptr, 2, st);
    const int adj_op = lsum ? SOP_ADJL : SOP_ADJ;
    const int adj_rop = lsum ? SOP_ADJLR : SOP_ADJR;
    int lam_first = 1;
    const void *lcur = lam_T;
    // A one-step advance whose result only the next adjoint step reads is
    // folded into that step: the adjoint kernel recomputes u_s at each point
    // from u_{s-1}, with the advance's arithmetic, instead of reading it.
    auto fold = [&](size_t i) {
        const RvOp &a = ops[i];
        if (a.kind != kRvAdvance || a.t1 - a.t0 != 1 || i + 1 >= ops.size()) return false;
        const RvOp &b = ops[i + 1];
        if (b.kind != kRvAdjoint || b.src != a.dst || b.t0 != a.t1) return false;
        for (size_t j = i + 2; j < ops.size(); ++j) {  // is the advance's buffer read again?
            if (ops[j].src == a.dst) return false;
            if (ops[j].kind == kRvAdvance && ops[j].dst == a.dst) break;
        }
        return true;
    };
    // A chain of one-step advances, each from the previous one's state into
    // a buffer of its own, is one pass of two or three steps that stores
    // every state it passes.
    auto chain = [&](size_t i) {
        size_t j = i;
        while (j + 1 < ops.size() && j - i < 2) {
            const RvOp &a = ops[j], &b = ops[j + 1];
            if (b.kind != kRvAdvance || b.t1 - b.t0 != 1 || b.src != a.dst || b.t0 != a.t1) break;
            bool fresh = b.dst != ops[i].src;
            for (size_t k = i; k <= j; ++k) fresh = fresh && ops[k].dst != b.dst;
            if (!fresh) break;
            ++j;
        }
        return j > i ? pp.len_at(0, (int32_t)(j - i + 1)) : 1;
    };
    // the opening chain of advances was run by dcp_revolve_forward
    size_t i0 = 0;
    while (i0 < ops.size() && ops[i0].kind == kRvAdvance) ++i0;
    for (size_t i = i0; i < ops.size(); ++i) {
        const RvOp &op = ops[i];
        if (op.kind == kRvAdvance && op.t1 - op.t0 == 1) {
            const int len = chain(i);
            if (len >= 2) {
                DCP_TRY(fwd_pass(dtype, bc, g, c, tf, pp, len, B.buf(op.src), f, B.buf(ops[i + len - 1].dst),
                                 B.buf(op.dst), len == 3 ? B.buf(ops[i + 1].dst) : nullptr, st));
                i += len - 1;
                continue;
            }
        }
        const bool folded = fold(i);
        if (op.kind == kRvAdvance && !folded) {
            if ((rc = rev_advance(dtype, bc, g, c, tf, pp, f, B.buf(op.src), B.buf(op.dst), scratch,
                                  op.t1 - op.t0, st)))
                return rc;
            continue;
        }
        // adjoint step s with u_s in buffer src, or recomputed from u_{s-1};
        // or steps s and s - 1 when the next operation is step s - 1
        const RvOp &adj = folded ? ops[i + 1] : op;
        const int32_t s = (int32_t)adj.t0;
        const bool pair = !folded && ap.nblk && i + 1 < ops.size() && ops[i + 1].kind == kRvAdjoint &&
                          ops[i + 1].t0 == s - 1;
        const int32_t se = pair ? s - 1 : s;
        DCP_TRY(step_sums.take(se, s + 1));
        void *out = (se == 0) ? grad_u0 : (lcur == lam[0] ? lam[1] : lam[0]);
        if (pair) {
            ta.u = lcur;
            ta.f = B.buf(adj.src);
            ta.g2 = B.buf(ops[i + 1].src);
            ta.out = out;
            ta.mid = nullptr;
            ta.part1 = step_sums.of(s);
            ta.part2 = step_sums.of(s - 1);
            ta.lam_first = lam_first;
            DCP_TRY(adj_pair(dtype, adj_op, bc, ap, ta, st));
            step_sums.set(s - 1, s + 1, ap.nblk);
        } else {
            aa.s = lcur;
            aa.q = folded ? f : B.buf(adj.src);
            aa.s2 = folded ? B.buf(op.src) : nullptr;
            aa.out = out;
            aa.partials = step_sums.of(s);
            aa.lam_first = lam_first;
            DCP_TRY(launch_stencil(dtype, folded ? adj_rop : adj_op, bc, true, t, aa, st));
        }
        lam_first = 0;
        lcur = out;
        if (folded || pair) ++i;
    }
    // per-step sums in a fixed order, then over the steps in a fixed order
    DCP_TRY(step_sums.reduce());
    DCP_TRY(launch_grad_finalize(sums, T, c.dt / (c.h * c.h), -c.dt, grad_ab, st));
    if (lsum) {
        if (grad_gamma) {
            double *dp = reinterpret_cast<double *>(at(ws, w.dot));
            const int nb = ew_norm_blocks(g.n);
            double *pair = dp + 2 * (size_t)nb;
            DCP_TRY(launch_ew_dot(dtype, lsum, f, dp, g.n, ew_ok({lsum, f}), st));
            DCP_TRY(launch_finalize(dp, nb, nb, 1, pair, nullptr, 0, st));
            DCP_TRY(launch_scalar_scale(pair, c.dt, grad_gamma, st));
        }
        if (grad_f)
            DCP_TRY(launch_ew(dtype, EW_SCALE, grad_f, nullptr, grad_f, c.gamma * c.dt, g.n,
                              ew_ok({grad_f}), st));
    }
    return DCP_OK;
}

}  // extern "C"
