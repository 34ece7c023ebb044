// Trajectory cost sampling and adjoints on gfx950.
//
// Sampling (the cost and height terms of the trajectory optimisation of
// Sec. III-E, Eq. (11)): a waypoint (x, y, z) on slice k contributes
//     f = C_k(x, y) + w_z (z - G_k(x, y) - d_ref)^2,
// with C_k, G_k cell-centred bilinear interpolations of c^T_k and e^G_k
// (clamped at the grid edge, zero slope across the clamp); the height term
// is dropped when a ground corner is missing; a trajectory sums its
// waypoints.  Waypoints with a non-finite coordinate or a slice outside
// [0, N) contribute nothing.
//
// Adjoints: bilinear weights scatter dL/dC and dL/dG to the four corners;
// the traversability adjoint routes dL/dc^T through the maximising tap of
// the Eq. (6) window (first maximum in row-major window order) into the
// Eq. (1)-(5) derivatives at that cell; the construction adjoint adds each
// ground/ceiling gradient to the z of the point that holds the value.  The
// maximising tap is found by recomputing c^init with the same FP32
// operation sequence as the forward kernels, so it reproduces the forward
// maximum exactly.
//
// Gradient sums: float atomics by default, whose result depends on the
// order in which the additions land; with PCT_FIXED_POINT, 64-bit integer
// atomics on contributions rounded to multiples of 2^-32, whose sum does
// not depend on that order (nor on how the work is split into launches).
#include <limits.h>

#include <utility>

#include "pct_internal.h"

namespace pct {

namespace {

constexpr int kBlock = 256;

__device__ __forceinline__ float sumsq(float dx, float dy) { return __builtin_fmaf(dx, dx, dy * dy); }

__device__ __forceinline__ float gval(const float* __restrict__ gk, int nx, int ny, int x, int y) {
    return (x >= 0 && y >= 0 && x < nx && y < ny) ? gk[(long long)y * nx + x] : -INFINITY;
}

// Where a cell's e^G and e^C come from: the map itself (off-grid cells have
// no ground), or a wavefront's staged box.
struct MapCells {
    const float* __restrict__ gk;
    const float* __restrict__ ck;
    int nx, ny;
    __device__ __forceinline__ float G(int x, int y) const { return gval(gk, nx, ny, x, y); }
    __device__ __forceinline__ float C(int x, int y) const { return ck[(long long)y * nx + x]; }
};

template <class Cells>
__device__ __forceinline__ bool gentle_at(const Cells& m, int x, int y, const EvalParams& p) {
    const float G = m.G(x, y);
    const float l = m.G(x - 1, y), r = m.G(x + 1, y);
    const float d = m.G(x, y - 1), u = m.G(x, y + 1);
    if (!(isfinite(G) && isfinite(l) && isfinite(r) && isfinite(d) && isfinite(u))) return false;
    return sumsq(r - l, u - d) < p.Ts2;
}

struct Cinit {
    float ci, dx, dy, dI;
    int branch;   // 0 no ground, 1 barrier, 2 gentle, 3 step, 4 step without support
    bool ipos;    // interval term active: d^I >= d_min and alpha_d (d_ref - d^I) > 0
    bool pass;    // c^I + c^G < c^B (the clip of Eq. (5) is not active)
};

// c^init of cell (x, y) of one slice, Eqs. (1)-(5), with the values needed
// by its adjoint.  Same FP32 operation sequence as the forward kernels.
template <class Cells>
__device__ __forceinline__ Cinit cinit_of(const Cells& m, int x, int y, float G, float C, const EvalParams& p) {
    Cinit o{};
    if (!isfinite(G)) {
        o.ci = p.cB;
        o.branch = 0;
        return o;
    }
    o.dI = C - G;
    const float cI = o.dI < p.d_min ? p.cB : fmaxf(0.0f, p.alpha_d * (p.d_ref - o.dI));
    o.ipos = !(o.dI < p.d_min) && p.alpha_d * (p.d_ref - o.dI) > 0.0f;
    const float l = m.G(x - 1, y), r = m.G(x + 1, y);
    const float d = m.G(x, y - 1), u = m.G(x, y + 1);
    float cG = p.cB;
    o.branch = 1;
    if (isfinite(l) && isfinite(r) && isfinite(d) && isfinite(u)) {
        o.dx = r - l;
        o.dy = u - d;
        if (!(fmaxf(fabsf(o.dx), fabsf(o.dy)) > p.Tb)) {
            const float s2 = sumsq(o.dx, o.dy);
            if (s2 < p.Ts2) {
                cG = p.As * s2;
                o.branch = 2;
            } else {
                int cnt = 0;
                for (int dyp = -p.rp; dyp <= p.rp; ++dyp)
                    for (int dxp = -p.rp; dxp <= p.rp; ++dxp)
                        if (dxp | dyp) cnt += gentle_at(m, x + dxp, y + dyp, p) ? 1 : 0;
                if (cnt > p.kp) {
                    cG = p.Ab * fmaxf(o.dx * o.dx, o.dy * o.dy);
                    o.branch = 3;
                } else {
                    o.branch = 4;
                }
            }
        }
    }
    const float s = cI + cG;
    o.pass = s < p.cB;
    o.ci = fminf(p.cB, s);
    return o;
}

__device__ __forceinline__ Cinit cinit_at(const float* __restrict__ gk, const float* __restrict__ ck, int x, int y,
                          const EvalParams& p) {
    const MapCells m{gk, ck, p.nx, p.ny};
    const float G = gk[(long long)y * p.nx + x];
    return cinit_of(m, x, y, G, isfinite(G) ? m.C(x, y) : 0.0f, p);
}

// A contribution in fixed point: v * 2^32 rounded to the nearest integer
// (ties to even), clamped to +-2^62 so that the conversion is defined; NaN
// adds nothing.
__device__ __forceinline__ unsigned long long to_fixed(float v) {
    const float q = rintf(v * 0x1p32f);
    if (!(q == q)) return 0ull;
    return (unsigned long long)(long long)fminf(fmaxf(q, -0x1p62f), 0x1p62f);
}

// Gradient sum: a float array, or with `fixed` an int64 array of 2^-32 units
// (two's complement, so integer addition wraps to the signed sum).
__device__ __forceinline__ void grad_add(float* p, long long i, float v, bool fixed) {
    if (fixed) atomicAdd((unsigned long long*)p + i, to_fixed(v));
    else atomicAdd(p + i, v);
}

// Gradient sink: dense grids (nullable) and/or point heights via the ids.
struct Sink {
    float* gG;          // [N][ny][nx] or null
    float* gC;          // [N][ny][nx] or null
    const int* aG;      // point ids, for routing to gz (null: no routing)
    const int* aC;
    float* gz;
    long long n_points;
    int fixed;          // the sums are int64 fixed point (gG, gC, gz)
};

__device__ __forceinline__ void add_ground(const Sink& s, long long i, float v) {
    if (v == 0.0f) return;
    if (s.gG) grad_add(s.gG, i, v, s.fixed);
    if (s.gz) {
        const int id = s.aG[i];
        if (id >= 0 && id < s.n_points) grad_add(s.gz, id, v, s.fixed);
    }
}
__device__ __forceinline__ void add_ceil(const Sink& s, long long i, float v) {
    if (v == 0.0f) return;
    if (s.gC) grad_add(s.gC, i, v, s.fixed);
    if (s.gz) {
        const int id = s.aC[i];
        if (id >= 0 && id < s.n_points) grad_add(s.gz, id, v, s.fixed);
    }
}

// c^T of cell (x, y) of one slice, evaluated on demand: the maximum over
// the Eq. (6) window of K * c^init (first maximum in row-major window
// order), with the maximising cell and its weight.  The same FP32
// products and maxima as the full-map kernels, so the same value.
struct WinMax {
    float v, k;
    int qx, qy;
};

// The window maxima of the four bilinear corners of a waypoint at once:
// corners (cx[c], cy[c]) lie in a 2 x 2 block, so their windows share most
// cells.  The union of the windows is walked once in row-major order,
// computing each cell's c^init once; every cell updates the corners whose
// window holds it.  Row-major order over the union is row-major order over
// each corner's window, so each corner gets the same first maximum as a walk
// over its own window.
__device__ void window_max4(const float* __restrict__ gk, const float* __restrict__ ck, const int (&cx)[4],
                            const int (&cy)[4], const EvalParams& p, WinMax (&o)[4]) {
    const int nx = p.nx, ny = p.ny, R = p.R;
    int xlo = cx[0], xhi = cx[0], ylo = cy[0], yhi = cy[0];
#pragma unroll
    for (int c = 1; c < 4; ++c) {
        xlo = min(xlo, cx[c]);
        xhi = max(xhi, cx[c]);
        ylo = min(ylo, cy[c]);
        yhi = max(yhi, cy[c]);
    }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        o[c] = WinMax{};
        o[c].v = -INFINITY;
    }
    for (int qy = max(0, ylo - R); qy <= min(ny - 1, yhi + R); ++qy) {
        for (int qx = max(0, xlo - R); qx <= min(nx - 1, xhi + R); ++qx) {
            bool need = false;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int m = abs(qx - cx[c]), n = abs(qy - cy[c]);
                need |= m <= R && n <= R && p.K[m][n] > 0.0f;
            }
            if (!need) continue;
            const float ci = cinit_at(gk, ck, qx, qy, p).ci;
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const int m = abs(qx - cx[c]), n = abs(qy - cy[c]);
                if (m > R || n > R) continue;
                const float kw = p.K[m][n];
                if (!(kw > 0.0f)) continue;
                const float v = kw * ci;
                if (v > o[c].v) {
                    o[c].v = v;
                    o[c].k = kw;
                    o[c].qx = qx;
                    o[c].qy = qy;
                }
            }
        }
    }
}

// LDS written by some lanes of a wavefront, then read by others.
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---------------------------------------------------------------- boxes
//
// A wavefront's box: the cells that the windows of its waypoints can touch
// on one slice.  e^G is staged in LDS with a halo of patch radius + 1 (one
// coalesced read per cell, -inf off the grid), c^init is evaluated from
// there once per cell (NaN off the grid), and the window maxima read only
// c^init.  With fixed-point sums the box also holds the ground gradients of
// its cells (integers, so the order of the additions does not matter), which
// go out in one atomic per touched cell when the wavefront leaves the box:
// atomics on device memory are what an adjoint that sends each contribution
// there by itself waits for.  64 profiles x 1024 walks x 256 waypoints on
// the 1000 x 1000 building, values and gradients: 12.5 ms with c^init
// evaluated from global memory and every contribution an atomic, 9.3 ms with
// boxes (7.7 ms of it the atomics), 2.8 ms with the box's sums and boxes kept
// from profile to profile; values alone 1.2 ms, bound by vector issue
// (3300 instructions per round of 64 waypoints).  LDS of 13 KB instead of
// 10 KB per wavefront cuts fewer groups but leaves three workgroups per CU:
// 3.1 ms, and 1.8 ms for the values alone.
constexpr int kBoxFloats = 2472;     // 4 workgroups of 4 wavefronts per CU
constexpr int kBoxR = 8;             // largest radius of a staged box; above, the weights take part of the box
constexpr int kBoxWeights = (kBoxR + 1) * (kBoxR + 1);
constexpr int kWideWeights = kKmax * kKmax;
struct BoxLds {
    // gradient sums, e^G with halo, c^init; then the weights K[a * (R + 1) + j],
    // NaN where zero
    alignas(8) float v[kBoxFloats + kBoxWeights + 1];
};
static_assert(4 * sizeof(BoxLds) * 4 <= 160 * 1024, "four workgroups per CU");

__device__ __forceinline__ int box_room(int R) {
    return R <= kBoxR ? kBoxFloats : kBoxFloats + kBoxWeights - kWideWeights;
}

struct Box {
    unsigned long long* acc;   // ground gradients, rows of w + 2 cells, first cell (x0 - 1, y0 - 1)
    float* g;                  // e^G, rows of wg cells, first cell (x0 - halo, y0 - halo)
    float* c;                  // c^init, rows of w cells, first cell (x0, y0)
    int x0, y0, w, h, wg, halo;
    int k;                     // slice; -1: nothing staged
    __device__ __forceinline__ float G(int x, int y) const { return g[(y - y0 + halo) * wg + x - x0 + halo]; }
};

// Whether a staged box of w x h cells fits (halo: patch radius + 1).
__host__ __device__ __forceinline__ bool box_fits(int w, int h, int halo, bool sums) {
    if (w > kBoxFloats || h > kBoxFloats) return false;
    const int e = 2 * halo;
    return (sums ? 2 * (w + 2) * (h + 2) : 0) + (w + e) * (h + e) + w * h <= kBoxFloats;
}

// Cells lane, lane + 64, ... of a row-major box `W` wide, without a division
// per cell.
struct BoxWalk {
    int u, v, du, dv, W;
    __device__ __forceinline__ BoxWalk(int lane, int W_) : W(W_) {
        v = lane / W;
        u = lane - v * W;
        dv = 64 / W;
        du = 64 - dv * W;
    }
    __device__ __forceinline__ void next() {
        u += du;
        v += dv;
        if (u >= W) {
            u -= W;
            ++v;
        }
    }
};

// The wavefront (all lanes) moves its box to the w x h cells at (x0, y0) of
// slice k: e^G staged four cells per lane and step, so that their loads are
// in flight together, gradient sums cleared.
__device__ __forceinline__ void stage_box(Box& b, BoxLds& lds, const float* __restrict__ gk, int k, int x0, int y0,
                                          int w, int h, const EvalParams& p, bool sums) {
    const int lane = threadIdx.x & 63, nx = p.nx, ny = p.ny;
    b.k = k;
    b.halo = p.rp + 1;
    b.x0 = x0;
    b.y0 = y0;
    b.w = w;
    b.h = h;
    b.wg = w + 2 * b.halo;
    const int ns = sums ? (w + 2) * (h + 2) : 0, n = b.wg * (h + 2 * b.halo);
    b.acc = (unsigned long long*)lds.v;
    b.g = lds.v + 2 * ns;
    b.c = b.g + n;
    for (int i = lane; i < ns; i += 64) b.acc[i] = 0ull;
    BoxWalk q(lane, b.wg);
    for (int i = lane; i < n; i += 256) {
        float v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[e] = i + 64 * e < n ? gval(gk, nx, ny, x0 - b.halo + q.u, y0 - b.halo + q.v) : 0.0f;
            q.next();
        }
#pragma unroll
        for (int e = 0; e < 4; ++e)
            if (i + 64 * e < n) b.g[i + 64 * e] = v[e];
    }
    wave_lds_sync();
}

// c^init of the box's cells for parameters p.
__device__ __forceinline__ void fill_cinit(const Box& b, const float* __restrict__ ck, const EvalParams& p) {
    const int lane = threadIdx.x & 63, nx = p.nx, ny = p.ny;
    BoxWalk q(lane, b.w);
    const int n = b.w * b.h;
    for (int i = lane; i < n; i += 256) {
        float C[4];
        int x[4], y[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            x[e] = b.x0 + q.u;
            y[e] = b.y0 + q.v;
            const bool in = i + 64 * e < n && x[e] >= 0 && y[e] >= 0 && x[e] < nx && y[e] < ny;
            C[e] = in ? ck[(long long)y[e] * nx + x[e]] : 0.0f;
            if (!in) x[e] = INT_MIN;
            q.next();
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (i + 64 * e >= n) continue;
            float ci = __builtin_nanf("");
            if (x[e] != INT_MIN) ci = cinit_of(b, x[e], y[e], b.G(x[e], y[e]), C[e], p).ci;
            b.c[i + 64 * e] = ci;
        }
    }
    wave_lds_sync();
}

// A box of c^init alone, w x h cells at (x0, y0), formed from the map.
__device__ __forceinline__ void bare_box(Box& b, BoxLds& lds, const float* __restrict__ gk,
                                         const float* __restrict__ ck, int x0, int y0, int w, int h,
                                         const EvalParams& p) {
    const int lane = threadIdx.x & 63;
    b.k = -1;
    b.x0 = x0;
    b.y0 = y0;
    b.w = w;
    b.h = h;
    b.c = lds.v;
    BoxWalk q(lane, w);
    for (int i = lane; i < w * h; i += 64) {
        const int x = x0 + q.u, y = y0 + q.v;
        float ci = __builtin_nanf("");
        if (x >= 0 && y >= 0 && x < p.nx && y < p.ny) ci = cinit_at(gk, ck, x, y, p).ci;
        b.c[i] = ci;
        q.next();
    }
    wave_lds_sync();
}

// The box's gradient sums to the sink (fixed point).
__device__ __forceinline__ void flush_box(const Box& b, const Sink& s, long long plane, int nx) {
    if (b.k < 0) return;
    wave_lds_sync();
    BoxWalk q(threadIdx.x & 63, b.w + 2);
    const int n = (b.w + 2) * (b.h + 2);
    for (int i = threadIdx.x & 63; i < n; i += 64) {
        const unsigned long long v = b.acc[i];
        if (v != 0ull) {
            const long long cell = (long long)b.k * plane + (long long)(b.y0 - 1 + q.v) * nx + (b.x0 - 1 + q.u);
            if (s.gG) atomicAdd((unsigned long long*)s.gG + cell, v);
            if (s.gz) {
                const int id = s.aG[cell];
                if (id >= 0 && id < s.n_points) atomicAdd((unsigned long long*)s.gz + id, v);
            }
        }
        q.next();
    }
    wave_lds_sync();
}

// Window maxima of the C2 x C2 corners (x + q, y + r), q, r < C2, corner
// r * C2 + q, from the box's c^init: per corner the first maximum of
// K * c^init in row-major window order, as a walk over its own window gives
// it.  Taps off the grid or of weight zero are NaN products, which fmaxf
// passes over and no comparison selects.  Each window row is reduced to its
// maximum and the first row with a greater one is remembered; the tap is
// then found in that row alone, when `taps` is set.  RT: the inflation radius
// when known at compile time, -1: p.R.
template <int RT, int C2>
__device__ __forceinline__ void window_max_box(const Box& b, const float* __restrict__ sK, int x, int y,
                                               const EvalParams& p, bool taps, WinMax (&o)[C2 * C2]) {
    constexpr int NC = C2 * C2;
    const int R = RT >= 0 ? RT : p.R, K1 = R + 1;
    const float* base = b.c + (y - R - b.y0) * b.w + (x - R - b.x0);
    float best[NC];
    int brow[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        best[c] = -INFINITY;
        brow[c] = 0;
    }
    if constexpr (RT >= 0) {
        constexpr int kRows = RT == 2 || RT == 4 || RT == 5 ? 2 * RT + C2 : 1;
#pragma unroll kRows
        for (int n = 0; n < 2 * RT + C2; ++n) {
            float v[2 * RT + C2];
#pragma unroll
            for (int m = 0; m < 2 * RT + C2; ++m) v[m] = base[n * b.w + m];
#pragma unroll
            for (int r = 0; r < C2; ++r) {
                const int dy = n - RT - r;
                if (dy < -RT || dy > RT) continue;   // uniform
                const int j = dy < 0 ? -dy : dy;
#pragma unroll
                for (int q = 0; q < C2; ++q) {
                    float rm = -INFINITY;
#pragma unroll
                    for (int m = 0; m <= 2 * RT; ++m)
                        rm = fmaxf(rm, sK[(m < RT ? RT - m : m - RT) * (RT + 1) + j] * v[m + q]);
                    const int c = C2 * r + q;
                    if (rm > best[c]) {
                        best[c] = rm;
                        brow[c] = n;
                    }
                }
            }
        }
    } else {
        for (int n = 0; n < 2 * R + C2; ++n) {
            float rm[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) rm[c] = -INFINITY;
            for (int m = 0; m < 2 * R + C2; ++m) {
                const float v = base[n * b.w + m];
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const int a = abs(m - R - c % C2), j = abs(n - R - c / C2);
                    if (a <= R && j <= R) rm[c] = fmaxf(rm[c], sK[a * K1 + j] * v);
                }
            }
#pragma unroll
            for (int c = 0; c < NC; ++c)
                if (rm[c] > best[c]) {
                    best[c] = rm[c];
                    brow[c] = n;
                }
        }
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        o[c] = WinMax{};
        o[c].v = best[c];
    }
    if (!taps) return;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int q = c % C2, r = c / C2;
        const int j = abs(brow[c] - R - r);
        const float* row = base + brow[c] * b.w + q;
        int bm = 0;
        float bk = 0.0f;
        for (int m = 2 * R; m >= 0; --m) {      // the last hit is the row's first maximum
            const float kw = sK[abs(m - R) * K1 + j];
            if (kw * row[m] == best[c]) {
                bm = m;
                bk = kw;
            }
        }
        o[c].k = bk;
        o[c].qx = x + q + bm - R;
        o[c].qy = y - R + brow[c];
    }
}

// How the radii's windows are walked: 2, 4 and 5 (the usual 0.3 m and the
// quadruped's 0.2 m of inflation on 0.1 m grids, and on 0.2 m) unrolled as a
// whole, 3 and 6 to 8 by unrolled rows, the others by run-time loops.  By rows
// the three take 5 to 10 % longer; more whole windows in one kernel spill its
// registers (64 profiles' kernel: 32 instead of 14), so the radii walked by
// rows and those above have kernels of their own.
__host__ __device__ constexpr bool wide_radius(int R) { return R == 3 || R > 5; }

// p.R is uniform over the wavefront.  WIDE: wide radii may come, else others.
template <int C2, bool NARROW, bool WIDE>
__device__ __forceinline__ void window_max_any(const Box& b, const float* __restrict__ sK, int x, int y,
                                               const EvalParams& p, bool taps, WinMax (&o)[C2 * C2]) {
#define PCT_W(RT)                                                        \
    if constexpr (wide_radius(RT) ? WIDE : NARROW)                       \
        if (p.R == RT) return window_max_box<RT, C2>(b, sK, x, y, p, taps, o);
    PCT_W(5) PCT_W(4) PCT_W(2) PCT_W(3) PCT_W(6) PCT_W(7) PCT_W(8)
#undef PCT_W
    window_max_box<-1, C2>(b, sK, x, y, p, taps, o);
}

// The wavefront's weight table for the parameters it works with.  Above
// kBoxR it takes part of the box: no staged box may be there.
__device__ __forceinline__ void fill_weights(BoxLds& lds, const EvalParams& p) {
    const int lane = threadIdx.x & 63, K1 = p.R + 1;
    float* K = lds.v + box_room(p.R);
    for (int i = lane; i < K1 * K1; i += 64) K[i] = p.K[i / K1][i % K1];
    wave_lds_sync();
}

// The window maxima of one waypoint's corners by the whole wavefront, from a
// box of its windows alone: every lane takes cells of the box, the maxima
// and their first taps are reduced over the lanes.
__device__ __forceinline__ void window_max4_one(const Box& b, const float* __restrict__ sK, const EvalParams& p,
                                                bool taps, WinMax (&o)[4]) {
    const int lane = threadIdx.x & 63, R = p.R, K1 = R + 1, n = b.w * b.h;
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const int q = c & 1, r = c >> 1;
        float best = -INFINITY, bk = 0.0f;
        int bi = INT_MAX;
        BoxWalk u(lane, b.w);
        for (int i = lane; i < n; i += 64) {
            const int m = abs(u.u - R - q), j = abs(u.v - R - r);
            const float kw = m <= R && j <= R ? sK[m * K1 + j] : __builtin_nanf("");
            const float v = kw * b.c[i];
            if (v > best) {
                best = v;
                bk = kw;
                bi = i;
            }
            u.next();
        }
        // c^init >= 0: the maximum is not negative, and the order of such
        // floats is that of their encodings
        const int top = wave_max_i(bi == INT_MAX ? -1 : __builtin_bit_cast(int, best));
        o[c] = WinMax{};
        o[c].v = __builtin_bit_cast(float, top);
        if (!taps) continue;
        const int first = wave_min_i(bi != INT_MAX && __builtin_bit_cast(int, best) == top ? bi : INT_MAX);
        o[c].k = __shfl(bk, first & 63, 64);      // cell i belongs to lane i % 64
        o[c].qy = b.y0 + first / b.w;
        o[c].qx = b.x0 + first % b.w;
    }
}

// Where a waypoint's gradients go: ground gradients to the box's sums when
// it has them, all others to the sink.
struct BoxSink {
    const Sink* s;
    const Box* b;      // null: no box sums
    long long base;    // first cell of the slice
    int nx;
    __device__ __forceinline__ void ground(int x, int y, float v) const {
        if (b) {
            if (v != 0.0f) atomicAdd(&b->acc[(y - b->y0 + 1) * (b->w + 2) + x - b->x0 + 1], to_fixed(v));
        } else {
            add_ground(*s, base + (long long)y * nx + x, v);
        }
    }
    __device__ __forceinline__ void ceil(int x, int y, float v) const {
        add_ceil(*s, base + (long long)y * nx + x, v);
    }
};

// The wavefront's waypoints in groups that share a box: `ok` lanes on slice
// k with corners (x, y) .. (x + 1, y + 1).  The lanes of the first waiting
// lane's slice, from it on, form a group; while their box does not fit, the
// group is cut to half its reach.  A group whose box lies in the one staged
// already (the next profile on the same walk) keeps it, with the gradients
// summed there; SUMS: the box sums ground gradients (fixed point), which leave
// with the box.  WIDE (wide_radius): a group that would be cut below
// 32 lanes, and any above kBoxR, takes a box of c^init alone for as many
// lanes as that holds, and its gradients go out one by one (256 walks x 256
// waypoints, radius 8: 2.02 ms with staged boxes of fewer than eight lanes
// and single waypoints, 0.38 so; radius 14: 8.06 ms by walks over the map, 1.30
// so).
// Groups of fewer than eight lanes would spend most of the wavefront on one
// window after another: those waypoints are taken one by one, the whole
// wavefront on each.  The weights of p are in place, and the map is more than
// one cell wide and tall.
// body(wm, detail, sink) runs once per lane, where detail(wm[c]) is the
// c^init of the maximising cell with what its adjoint needs.
template <bool SUMS, bool WIDE, class Body>
__device__ __forceinline__ void for_box_groups(Box& b, BoxLds& lds, const float* __restrict__ ground,
                                               const float* __restrict__ ceil, const EvalParams& p, bool ok, int k,
                                               int x, int y, bool taps, const Sink& s, Body body) {
    const int lane = threadIdx.x & 63, R = p.R, room = WIDE ? box_room(R) : kBoxFloats;
    const float* sK = lds.v + room;
    unsigned long long rem = __ballot(ok);
    while (rem != 0ull) {
        const int l0 = (int)__builtin_ctzll(rem);
        const int kb = __builtin_amdgcn_readlane(k, l0);
        const float* gk = ground + (long long)kb * p.plane;
        const float* ck = ceil + (long long)kb * p.plane;
        const bool cand = ((rem >> lane) & 1ull) != 0ull && k == kb;
        bool mine = false, fits = false, bare = false;
        int x0 = 0, y0 = 0, w = 0, h = 0;
        if constexpr (!WIDE) {
            for (int reach = 64; reach >= 8 && !fits; reach >>= 1) {
                mine = cand && lane < l0 + reach;
                x0 = wave_min_i(mine ? x : INT_MAX) - R;
                y0 = wave_min_i(mine ? y : INT_MAX) - R;
                w = wave_max_i(mine ? x : INT_MIN) + 2 + R - x0;
                h = wave_max_i(mine ? y : INT_MIN) + 2 + R - y0;
                fits = box_fits(w, h, p.rp + 1, SUMS);
            }
        } else {
            auto group = [&](int reach) {
                mine = cand && lane < l0 + reach;
                x0 = wave_min_i(mine ? x : INT_MAX) - R;
                y0 = wave_min_i(mine ? y : INT_MAX) - R;
                w = wave_max_i(mine ? x : INT_MIN) + 2 + R - x0;
                h = wave_max_i(mine ? y : INT_MIN) + 2 + R - y0;
            };
            for (int reach = 64; reach >= 32 && !fits && R <= kBoxR; reach >>= 1) {
                group(reach);
                fits = box_fits(w, h, p.rp + 1, SUMS);
            }
            for (int reach = 64; reach >= 8 && !fits && !bare; reach >>= 1) {
                group(reach);
                bare = w <= room && h <= room && w * h <= room;
            }
        }
        WinMax wm[4];
        if (fits || bare) {   // bare: WIDE only
            const bool staged = fits && b.k == kb && b.halo == p.rp + 1 && x0 >= b.x0 && y0 >= b.y0 &&
                                x0 + w <= b.x0 + b.w && y0 + h <= b.y0 + b.h;
            if (!staged) {
                if (SUMS) flush_box(b, s, p.plane, p.nx);
                if (!WIDE || fits) stage_box(b, lds, gk, kb, x0, y0, w, h, p, SUMS);
                else bare_box(b, lds, gk, ck, x0, y0, w, h, p);
            }
            if (!WIDE || fits) fill_cinit(b, ck, p);
            if (mine) window_max_any<2, !WIDE, WIDE>(b, sK, x, y, p, taps, wm);
        } else {
            if (SUMS) flush_box(b, s, p.plane, p.nx);
            unsigned long long left = __ballot(mine);
#pragma unroll
            for (int c = 0; c < 4; ++c) wm[c] = WinMax{};
            while (left != 0ull) {
                const int l = (int)__builtin_ctzll(left);
                WinMax one[4];
                const int xl = __builtin_amdgcn_readlane(x, l) - R, yl = __builtin_amdgcn_readlane(y, l) - R;
                if (!WIDE || R <= kBoxR) {
                    stage_box(b, lds, gk, kb, xl, yl, 2 + 2 * R, 2 + 2 * R, p, false);
                    fill_cinit(b, ck, p);
                } else {
                    bare_box(b, lds, gk, ck, xl, yl, 2 + 2 * R, 2 + 2 * R, p);
                }
                window_max4_one(b, sK, p, taps, one);
                wave_lds_sync();
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (lane == l) wm[c] = one[c];
                left &= left - 1;
            }
            b.k = -1;
        }
        if (mine) {
            const BoxSink to{&s, SUMS && fits ? &b : nullptr, (long long)kb * p.plane, p.nx};
            body(wm, [&](const WinMax& m) {
                const float C = ck[(long long)m.qy * p.nx + m.qx];
                if (fits) return cinit_of(b, m.qx, m.qy, b.G(m.qx, m.qy), C, p);
                return cinit_at(gk, ck, m.qx, m.qy, p);
            }, to);
        }
        wave_lds_sync();   // the next group refills the box
        rem &= ~__ballot(mine);
    }
}

// Eq. (1)-(5) adjoint at the maximising cell (x, y) of a window, for
// gradient gq of its c^init.
__device__ __forceinline__ void cinit_adjoint(const Cinit& q, int x, int y, float gq, const EvalParams& p,
                                              const BoxSink& to) {
    if (q.branch == 0 || !q.pass) return;
    if (q.ipos) {
        to.ground(x, y, p.alpha_d * gq);
        to.ceil(x, y, -p.alpha_d * gq);
    }
    float ddx = 0.0f, ddy = 0.0f;   // dL/d(dx), dL/d(dy) for the raw differences
    if (q.branch == 2) {
        ddx = 2.0f * p.As * q.dx * gq;
        ddy = 2.0f * p.As * q.dy * gq;
    } else if (q.branch == 3) {
        if (fabsf(q.dx) >= fabsf(q.dy)) ddx = 2.0f * p.Ab * q.dx * gq;
        else ddy = 2.0f * p.Ab * q.dy * gq;
    }
    if (ddx != 0.0f) {
        to.ground(x + 1, y, ddx);
        to.ground(x - 1, y, -ddx);
    }
    if (ddy != 0.0f) {
        to.ground(x, y + 1, ddy);
        to.ground(x, y - 1, -ddy);
    }
}

// dL/dc^T(k, x, y) = gc: inflation argmax, then the Eq. (1)-(5) adjoint.
__device__ void eval_adjoint_cell(const float* __restrict__ ground, const float* __restrict__ ceil, int k, int x,
                                  int y, float gc, const EvalParams& p, const Sink& s) {
    const long long base = (long long)k * p.plane;
    const float* gk = ground + base;
    const float* ck = ceil + base;
    const int nx = p.nx, ny = p.ny, R = p.R;
    float best = -INFINITY, bk = 0.0f;
    int bx = x, by = y;
    for (int n = -R; n <= R; ++n) {
        const int qy = y + n;
        if (qy < 0 || qy >= ny) continue;
        for (int m = -R; m <= R; ++m) {
            const int qx = x + m;
            const float kw = p.K[abs(m)][abs(n)];
            if (!(kw > 0.0f) || qx < 0 || qx >= nx) continue;
            const float v = kw * cinit_at(gk, ck, qx, qy, p).ci;
            if (v > best) {
                best = v;
                bk = kw;
                bx = qx;
                by = qy;
            }
        }
    }
    cinit_adjoint(cinit_at(gk, ck, bx, by, p), bx, by, bk * gc, p, BoxSink{&s, nullptr, base, nx});
}

// ----------------------------------------------------------------- sampling
struct SampleArgs {
    float x0, y0, res, inv_res, d_ref, w_z;
    int nx, ny, N;
    long long plane;
    int T, W;
};

struct Bil {
    bool ok, hterm;
    int i0, j0;       // cell of c00; the other corners are one further (the same cell on an axis of one cell)
    long long c00, c10, c01, c11;
    float fu, fv, du, dv;
};

// Cell-centred coordinate u = (x - x0) / r - 1/2 split into an integer
// part and a fraction.  Far from the origin u is large (2000 cells on a
// 200 m map) and one FP32 rounding of u would cost ~1e-4 of a cell; here
// the subtraction's error (two-sum) and the exact remainder of the
// correctly rounded quotient, fma(-q, r, dx), give the fraction to ~1e-7.
__device__ __forceinline__ void split_coord(float x, float x0, float r, int& i, float& f) {
    // dx + e = x - x0 exactly (two-sum)
    const float dx = x - x0;
    const float bb = dx - x;
    const float e = (x - (dx - bb)) + (-x0 - bb);
    const float q = dx / r;
    const float rem = __builtin_fmaf(-q, r, dx) + e;
    const float qs = q - 0.5f;
    const float fl = floorf(qs);
    f = (qs - fl) + rem / r;
    i = (int)fl;
    if (f < 0.0f) { f += 1.0f; --i; }
    else if (f >= 1.0f) { f -= 1.0f; ++i; }
}

// Clamp to the grid edge (zero slope across the clamp): u = i + f.
__device__ __forceinline__ void axis(int i, float f, int n, int& i0, int& i1, float& fr, float& dq) {
    if (n == 1) {
        i0 = i1 = 0;
        fr = 0.0f;
        dq = 0.0f;
        return;
    }
    dq = 1.0f;
    if (i < 0) {                                   // u < 0
        i = 0;
        f = 0.0f;
        dq = 0.0f;
    } else if (i > n - 1 || (i == n - 1 && f > 0.0f)) {   // u > n - 1
        i = n - 1;
        f = 0.0f;
        dq = 0.0f;
    }
    if (i > n - 2) {                               // u = n - 1 exactly
        i = n - 2;
        f += 1.0f;
    }
    i0 = i;
    i1 = i + 1;
    fr = f;
}

__device__ Bil bilinear(const float* __restrict__ ground, const SampleArgs& a, float x, float y, float z, int k) {
    Bil b{};
    if (k < 0 || k >= a.N || !isfinite(x) || !isfinite(y) || !isfinite(z)) return b;
    b.ok = true;
    int iu, iv, i0, i1, j0, j1;
    float fu, fv;
    split_coord(x, a.x0, a.res, iu, fu);
    split_coord(y, a.y0, a.res, iv, fv);
    axis(iu, fu, a.nx, i0, i1, b.fu, b.du);
    axis(iv, fv, a.ny, j0, j1, b.fv, b.dv);
    b.du *= a.inv_res;
    b.dv *= a.inv_res;
    b.i0 = i0;
    b.j0 = j0;
    const long long base = (long long)k * a.plane;
    b.c00 = base + (long long)j0 * a.nx + i0;
    b.c10 = base + (long long)j0 * a.nx + i1;
    b.c01 = base + (long long)j1 * a.nx + i0;
    b.c11 = base + (long long)j1 * a.nx + i1;
    b.hterm = isfinite(ground[b.c00]) && isfinite(ground[b.c10]) && isfinite(ground[b.c01]) && isfinite(ground[b.c11]);
    return b;
}

__global__ __launch_bounds__(kBlock) void k_sample_fwd(const float* __restrict__ cost, const float* __restrict__ ground,
                                                       const float* __restrict__ wp, const int* __restrict__ slice,
                                                       SampleArgs a, float* __restrict__ f) {
    const int t = blockIdx.x * (kBlock / 64) + (int)(threadIdx.x / 64);
    if (t >= a.T) return;
    const int lane = threadIdx.x & 63;
    float acc = 0.0f;
    for (int w = lane; w < a.W; w += 64) {
        const long long i = (long long)t * a.W + w;
        const float x = wp[3 * i], y = wp[3 * i + 1], z = wp[3 * i + 2];
        const Bil b = bilinear(ground, a, x, y, z, slice[i]);
        if (!b.ok) continue;
        const float w00 = (1.0f - b.fu) * (1.0f - b.fv), w10 = b.fu * (1.0f - b.fv);
        const float w01 = (1.0f - b.fu) * b.fv, w11 = b.fu * b.fv;
        acc += w00 * cost[b.c00] + w10 * cost[b.c10] + w01 * cost[b.c01] + w11 * cost[b.c11];
        if (b.hterm) {
            const float G = w00 * ground[b.c00] + w10 * ground[b.c10] + w01 * ground[b.c01] + w11 * ground[b.c11];
            const float e = z - G - a.d_ref;
            acc += a.w_z * e * e;
        }
    }
    for (int m = 32; m >= 1; m >>= 1) acc += __shfl_xor(acc, m, 64);
    if (lane == 0) f[t] = acc;
}

// Per waypoint: dL/dwp (written), the bilinear scatter of dL/dC to c^T
// (dense gcost) or, with EVAL, straight through the traversability adjoint
// into the sink, and of the height term to e^G.  With EVAL = kBoxes a
// wavefront's 64 waypoints share boxes of c^init as in k_traj_value_grad
// (kWideBoxes for wide radii); kWindows walks each corner's window over the map (maps that boxes do
// not take).
enum { kDense, kBoxes, kWideBoxes, kWindows };
template <int EVAL>
__global__ __launch_bounds__(kBlock, 4) void k_sample_bwd(const float* __restrict__ cost, const float* __restrict__ ground,
                                                       const float* __restrict__ ceil, const float* __restrict__ wp,
                                                       const int* __restrict__ slice, SampleArgs a,
                                                       const float* __restrict__ gf, float* __restrict__ gwp,
                                                       float* __restrict__ gcost, const EvalParams ep, Sink s) {
    const long long n = (long long)a.T * a.W;
    const long long i0 = (long long)blockIdx.x * kBlock + threadIdx.x;
    const bool act = i0 < n;
    if (EVAL == kDense && !act) return;
    const long long i = act ? i0 : n - 1;
    const int t = (int)(i / a.W);
    const float x = wp[3 * i], y = wp[3 * i + 1], z = wp[3 * i + 2];
    const int k = slice[i];
    Bil b = bilinear(ground, a, x, y, z, k);
    b.ok = b.ok && act;
    float gx = 0.0f, gy = 0.0f, gzw = 0.0f, g = 0.0f;
    float ws[4] = {0.0f, 0.0f, 0.0f, 0.0f};
    if (b.ok) {
        g = gf[t];
        const float w00 = (1.0f - b.fu) * (1.0f - b.fv), w10 = b.fu * (1.0f - b.fv);
        const float w01 = (1.0f - b.fu) * b.fv, w11 = b.fu * b.fv;
        const float c00 = cost[b.c00], c10 = cost[b.c10], c01 = cost[b.c01], c11 = cost[b.c11];
        const float dCdu = (1.0f - b.fv) * (c10 - c00) + b.fv * (c11 - c01);
        const float dCdv = (1.0f - b.fu) * (c01 - c00) + b.fu * (c11 - c10);
        gx = g * dCdu * b.du;
        gy = g * dCdv * b.dv;
        const long long cs[4] = {b.c00, b.c10, b.c01, b.c11};
        ws[0] = w00, ws[1] = w10, ws[2] = w01, ws[3] = w11;
        if (b.hterm) {
            const float G00 = ground[b.c00], G10 = ground[b.c10], G01 = ground[b.c01], G11 = ground[b.c11];
            const float G = w00 * G00 + w10 * G10 + w01 * G01 + w11 * G11;
            const float de = 2.0f * a.w_z * (z - G - a.d_ref) * g;
            const float dGdu = (1.0f - b.fv) * (G10 - G00) + b.fv * (G11 - G01);
            const float dGdv = (1.0f - b.fu) * (G01 - G00) + b.fu * (G11 - G10);
            gx -= de * dGdu * b.du;
            gy -= de * dGdv * b.dv;
            gzw = de;
            for (int c = 0; c < 4; ++c) add_ground(s, cs[c], -de * ws[c]);
        }
        for (int c = 0; c < 4; ++c) {
            const float gc = g * ws[c];
            if (gcost && gc != 0.0f) grad_add(gcost, cs[c], gc, s.fixed);
            if (EVAL == kWindows && gc != 0.0f) {
                const long long local = cs[c] - (long long)k * a.plane;
                eval_adjoint_cell(ground, ceil, k, (int)(local % a.nx), (int)(local / a.nx), gc, ep, s);
            }
        }
    }
    if (act) {
        gwp[3 * i] = gx;
        gwp[3 * i + 1] = gy;
        gwp[3 * i + 2] = gzw;
    }
    if constexpr (EVAL == kBoxes || EVAL == kWideBoxes) {
        __shared__ BoxLds s_box[kBlock / 64];
        BoxLds& lds = s_box[threadIdx.x / 64];
        fill_weights(lds, ep);
        Box box{};
        box.k = -1;
        auto body = [&](const WinMax (&wm)[4], auto detail, const BoxSink& to) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const float gc = g * ws[c];
                if (gc == 0.0f) continue;
                cinit_adjoint(detail(wm[c]), wm[c].qx, wm[c].qy, wm[c].k * gc, ep, to);
            }
        };
        const bool ok = b.ok && g != 0.0f;
        if (s.fixed) {
            for_box_groups<true, EVAL == kWideBoxes>(box, lds, ground, ceil, ep, ok, k, b.i0, b.j0, true, s, body);
            flush_box(box, s, a.plane, a.nx);
        } else {
            for_box_groups<false, EVAL == kWideBoxes>(box, lds, ground, ceil, ep, ok, k, b.i0, b.j0, true, s, body);
        }
    }
}

// Dense traversability adjoint, one thread per cell-slice with a gradient:
// for radii and patches whose windows no box holds.
__global__ __launch_bounds__(kBlock) void k_eval_bwd(const float* __restrict__ ground, const float* __restrict__ ceil,
                                                     const float* __restrict__ gcost, const EvalParams p, Sink s) {
    const long long total = p.plane * p.N;
    for (long long i = (long long)blockIdx.x * kBlock + threadIdx.x; i < total;
         i += (long long)gridDim.x * kBlock) {
        const float gc = gcost[i];
        if (gc == 0.0f) continue;
        const int k = (int)(i / p.plane);
        const long long c = i - (long long)k * p.plane;
        eval_adjoint_cell(ground, ceil, k, (int)(c % p.nx), (int)(c / p.nx), gc, p, s);
    }
}

// The same by tiles of tw x th cells (tw a power of two at most 64, th rows),
// a wavefront at a time: tiles without a gradient are passed over, the others
// form c^init of their windows once in a box.  A wavefront looks over
// kEvalLook rows of 64 columns at once (64 / tw tiles side by side), so that
// the mostly empty gradient grid streams.  One thread per cell walking its
// window over the map evaluated c^init (2 R + 1)^2 times per cell: a
// gradient step through 1024 walks on 500 x 500 x 57 cell-slices took 1.54
// ms, of which 0.72 ms there, against 0.86 ms with tiles and k_route's wider
// loads.
// KIND: kWideTiles takes wide radii, kLoneTiles those up to kEvalWalkR, kTiles
// the others.  kLoneTiles: where a strip of 64 columns holds at most kEvalWalk
// gradients, no two in one column, each lane walks the nine cells of its
// window over the map instead: a box of 180 values for each lone cell took
// longer.  400 x 400 x 51 cell-slices at radius 1, walked throughout / boxes
// throughout / this rule: a gradient at 0.3 % of the cells 168 / 214 / 175 us,
// at 1 % 270 / 278 / 241, at 3 % 374 / 320 / 320, at all 1123 / 352 / 350.
// At radius 2 the boxes are level at 0.1 % and faster above it.
constexpr int kEvalLook = 8;
constexpr int kEvalWalkR = 1, kEvalWalk = 10;
enum { kTiles, kWideTiles, kLoneTiles };

template <bool SUMS, int KIND>
__global__ __launch_bounds__(kBlock, 4) void k_eval_bwd_tiles(const float* __restrict__ ground,
                                                              const float* __restrict__ ceil,
                                                              const float* __restrict__ gcost, const EvalParams p,
                                                              int tw, int th, int nbx, int nby, Sink s) {
    __shared__ BoxLds s_box[kBlock / 64];
    BoxLds& lds = s_box[threadIdx.x / 64];
    fill_weights(lds, p);
    const float* sK = lds.v + kBoxFloats;
    const int lane = threadIdx.x & 63, R = p.R;
    const long long n_work = (long long)nbx * nby * p.N;
    const long long stride = (long long)gridDim.x * (kBlock / 64);
    for (long long wk = (long long)blockIdx.x * (kBlock / 64) + threadIdx.x / 64; wk < n_work; wk += stride) {
        const int k = __builtin_amdgcn_readfirstlane((int)(wk / ((long long)nbx * nby)));
        const int r = __builtin_amdgcn_readfirstlane((int)(wk % ((long long)nbx * nby)));
        const int X0 = r % nbx * 64, Y0 = r / nbx * kEvalLook;
        const float* gk = ground + (long long)k * p.plane;
        const float* ck = ceil + (long long)k * p.plane;
        const float* qk = gcost + (long long)k * p.plane;
        float v[kEvalLook];
#pragma unroll
        for (int e = 0; e < kEvalLook; ++e) {
            const int x = X0 + lane, y = Y0 + e;
            v[e] = x < p.nx && y < p.ny ? qk[(long long)y * p.nx + x] : 0.0f;
        }
        unsigned rows = 0u;   // rows in which this lane's column has a gradient (NaN included)
#pragma unroll
        for (int e = 0; e < kEvalLook; ++e) rows |= v[e] != 0.0f ? 1u << e : 0u;
        if (KIND == kLoneTiles && __popcll(__ballot(rows != 0u)) <= kEvalWalk &&
            __ballot((rows & (rows - 1u)) != 0u) == 0ull) {
            if (rows != 0u) {
                const int y = Y0 + __builtin_ctz(rows);
                eval_adjoint_cell(ground, ceil, k, X0 + lane, y, qk[(long long)y * p.nx + X0 + lane], p, s);
            }
            continue;
        }
        for (int ty = 0; ty < kEvalLook; ty += th) {
            unsigned long long cols = __ballot(((rows >> ty) & ((1u << th) - 1u)) != 0u);
            while (cols != 0ull) {
                const int tx = (int)__builtin_ctzll(cols) & ~(tw - 1);
                cols &= ~((tw == 64 ? ~0ull : (1ull << tw) - 1ull) << tx);
                const int x0 = X0 + tx, y0 = Y0 + ty;
                Box b{};
                stage_box(b, lds, gk, k, x0 - R, y0 - R, tw + 2 * R, th + 2 * R, p, SUMS);
                fill_cinit(b, ck, p);
                for (int c = lane; c < tw * th; c += 64) {
                    const int x = x0 + (c & (tw - 1)), y = y0 + c / tw;
                    const float gc = x < p.nx && y < p.ny ? qk[(long long)y * p.nx + x] : 0.0f;
                    if (gc == 0.0f) continue;
                    WinMax m[1];
                    window_max_any<1, KIND != kWideTiles, KIND == kWideTiles>(b, sK, x, y, p, true, m);
                    const float C = ck[(long long)m[0].qy * p.nx + m[0].qx];
                    const BoxSink to{&s, SUMS ? &b : nullptr, (long long)k * p.plane, p.nx};
                    cinit_adjoint(cinit_of(b, m[0].qx, m[0].qy, b.G(m[0].qx, m[0].qy), C, p), m[0].qx, m[0].qy,
                                  m[0].k * gc, p, to);
                }
                if (SUMS) flush_box(b, s, p.plane, p.nx);
                else wave_lds_sync();   // the next tile refills the box
            }
        }
    }
}

// Construction adjoint: per cell, walk the slices and add each run of
// values held by the same point in one atomic.  The ids and gradients of
// eight slices are loaded together: read one slice at a time the walk waited
// for each (500 x 500 x 57 slices, ground and ceiling: 126 us).
__global__ __launch_bounds__(kBlock) void k_route(const float* __restrict__ gG, const float* __restrict__ gC,
                                                  const int* __restrict__ aG, const int* __restrict__ aC,
                                                  long long plane, int N, long long n_points, float* __restrict__ gz,
                                                  int fixed) {
    const long long c = (long long)blockIdx.x * kBlock + threadIdx.x;
    if (c >= plane) return;
    constexpr int kAhead = 8;
    for (int which = 0; which < 2; ++which) {
        const float* g = which ? gC : gG;
        const int* a = which ? aC : aG;
        if (!g) continue;
        int cur = -1;
        float acc = 0.0f;
        for (int k0 = 0; k0 < N; k0 += kAhead) {
            int id[kAhead];
            float v[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const long long i = (long long)min(k0 + u, N - 1) * plane + c;
                id[u] = a[i];
                v[u] = g[i];
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                if (k0 + u >= N) break;
                if (id[u] != cur) {
                    if (cur >= 0 && cur < n_points && acc != 0.0f) grad_add(gz, cur, acc, fixed);
                    cur = id[u];
                    acc = 0.0f;
                }
                acc += v[u];
            }
        }
        if (cur >= 0 && cur < n_points && acc != 0.0f) grad_add(gz, cur, acc, fixed);
    }
}

// Fixed-point sums to float32: the integer correctly rounded, times 2^-32.
__global__ __launch_bounds__(kBlock) void k_fixed_to_float(const long long* __restrict__ q, long long n,
                                                           float* __restrict__ out) {
    for (long long i = (long long)blockIdx.x * kBlock + threadIdx.x; i < n; i += (long long)gridDim.x * kBlock)
        out[i] = (float)q[i] * 0x1p-32f;
}

__global__ __launch_bounds__(kBlock) void k_zero(float* __restrict__ p, long long n) {
    for (long long i = (long long)blockIdx.x * kBlock + threadIdx.x; i < n; i += (long long)gridDim.x * kBlock)
        p[i] = 0.0f;
}

int grid_for(long long n) { return (int)std::max<long long>(1, std::min<long long>((n + kBlock - 1) / kBlock, 1 << 16)); }

// Value and gradient for many robot profiles in one launch, each profile
// with its own trajectories, with c^T evaluated on demand at the bilinear
// corners (no cost maps).  One wavefront per trajectory and run of up to
// kTrajProfiles profiles, lanes over its waypoints: per round of 64
// waypoints the profiles follow one another, so that profiles on the same
// walk share the round's box.  Per waypoint the value and the waypoint
// gradient are the same FP32 sequences as k_sample_fwd / k_sample_bwd on a
// materialised map, and the maximising taps found for the value feed the
// traversability adjoint directly.
// SUMS: fixed-point gradient sums with a ground or point output.
// BOX: kWideBoxes takes the profiles of wide radii, kBoxes the others (a call
// with both launches both); kWindows walks the windows of all over
// the map, one profile per wavefront (maps that boxes do not take).
constexpr int kTrajProfiles = 8;

template <int BOX>
__device__ __forceinline__ bool takes_radius(int R) {
    return BOX == kWindows || wide_radius(R) == (BOX == kWideBoxes);
}

template <int BOX, bool SUMS>
__global__ __launch_bounds__(kBlock, 4) void k_traj_value_grad(const float* __restrict__ ground,
                                                               const float* __restrict__ ceil,
                                                               const EvalParams* __restrict__ robots, SampleArgs a,
                                                               int n_profiles, int run, const float* __restrict__ wp,
                                                               const int* __restrict__ slice,
                                                               const float* __restrict__ gf, float* __restrict__ f,
                                                               float* __restrict__ gwp, Sink s) {
    const long long wave = (long long)blockIdx.x * (kBlock / 64) + threadIdx.x / 64;
    const int p0 = __builtin_amdgcn_readfirstlane((int)(wave / a.T)) * run;
    const int t = __builtin_amdgcn_readfirstlane((int)(wave % a.T));
    if (p0 >= n_profiles) return;
    const int np = min(run, n_profiles - p0);
    const int lane = threadIdx.x & 63;
    __shared__ BoxLds s_box[BOX != kWindows ? kBlock / 64 : 1];
    BoxLds& lds = s_box[BOX != kWindows ? threadIdx.x / 64 : 0];
    Box box{};
    box.k = -1;
    int weights_of = -1;
    float accs[kTrajProfiles];
#pragma unroll
    for (int q = 0; q < kTrajProfiles; ++q) accs[q] = 0.0f;
    for (int w0 = 0; w0 < a.W; w0 += 64) {
        for (int pi = 0; pi < np; ++pi) {
            const EvalParams& p = robots[p0 + pi];
            if (!takes_radius<BOX>(p.R)) continue;   // uniform
            const long long row = (long long)(p0 + pi) * a.T + t;
            const int w = w0 + lane;
            const bool act = w < a.W;
            const long long i = row * a.W + min(w, a.W - 1);
            const float x = wp[3 * i], y = wp[3 * i + 1], z = wp[3 * i + 2];
            const int k = slice[i];
            const float g = gf ? gf[row] : 0.0f;
            Bil b = bilinear(ground, a, x, y, z, k);
            b.ok = b.ok && act;
            float gx = 0.0f, gy = 0.0f, gzw = 0.0f;
            float acc = 0.0f;
#pragma unroll
            for (int q = 0; q < kTrajProfiles; ++q) acc = q == pi ? accs[q] : acc;
            auto body = [&](const WinMax (&wm)[4], auto detail, const BoxSink& to) {
                const float w00 = (1.0f - b.fu) * (1.0f - b.fv), w10 = b.fu * (1.0f - b.fv);
                const float w01 = (1.0f - b.fu) * b.fv, w11 = b.fu * b.fv;
                const float ws[4] = {w00, w10, w01, w11};
                acc += w00 * wm[0].v + w10 * wm[1].v + w01 * wm[2].v + w11 * wm[3].v;
                float G00 = 0.0f, G10 = 0.0f, G01 = 0.0f, G11 = 0.0f, G = 0.0f;
                if (b.hterm) {
                    G00 = ground[b.c00];
                    G10 = ground[b.c10];
                    G01 = ground[b.c01];
                    G11 = ground[b.c11];
                    G = w00 * G00 + w10 * G10 + w01 * G01 + w11 * G11;
                    const float e = z - G - p.d_ref;
                    acc += a.w_z * e * e;
                }
                if (!gf) return;
                const float dCdu = (1.0f - b.fv) * (wm[1].v - wm[0].v) + b.fv * (wm[3].v - wm[2].v);
                const float dCdv = (1.0f - b.fu) * (wm[2].v - wm[0].v) + b.fu * (wm[3].v - wm[1].v);
                gx = g * dCdu * b.du;
                gy = g * dCdv * b.dv;
                if (b.hterm) {
                    const float de = 2.0f * a.w_z * (z - G - p.d_ref) * g;
                    const float dGdu = (1.0f - b.fv) * (G10 - G00) + b.fv * (G11 - G01);
                    const float dGdv = (1.0f - b.fu) * (G01 - G00) + b.fu * (G11 - G10);
                    gx -= de * dGdu * b.du;
                    gy -= de * dGdv * b.dv;
                    gzw = de;
                    const int x1 = min(b.i0 + 1, a.nx - 1), y1 = min(b.j0 + 1, a.ny - 1);
                    to.ground(b.i0, b.j0, -de * ws[0]);
                    to.ground(x1, b.j0, -de * ws[1]);
                    to.ground(b.i0, y1, -de * ws[2]);
                    to.ground(x1, y1, -de * ws[3]);
                }
#pragma unroll
                for (int c = 0; c < 4; ++c) {
                    const float gc = g * ws[c];
                    if (gc == 0.0f) continue;
                    cinit_adjoint(detail(wm[c]), wm[c].qx, wm[c].qy, wm[c].k * gc, p, to);
                }
            };
            if constexpr (BOX != kWindows) {
                if (weights_of != pi) {
                    if (BOX == kWideBoxes && p.R > kBoxR) {
                        if (SUMS) flush_box(box, s, a.plane, a.nx);
                        box.k = -1;
                    }
                    fill_weights(lds, p);
                    weights_of = pi;
                }
                for_box_groups<SUMS, BOX == kWideBoxes>(box, lds, ground, ceil, p, b.ok, k, b.i0, b.j0, gf != nullptr, s, body);
            } else if (b.ok) {
                const float* gk = ground + (long long)k * a.plane;
                const float* ck = ceil + (long long)k * a.plane;
                const int x1 = min(b.i0 + 1, a.nx - 1), y1 = min(b.j0 + 1, a.ny - 1);
                const int cx[4] = {b.i0, x1, b.i0, x1}, cy[4] = {b.j0, b.j0, y1, y1};
                WinMax wm[4];
                window_max4(gk, ck, cx, cy, p, wm);
                body(wm, [&](const WinMax& m) { return cinit_at(gk, ck, m.qx, m.qy, p); },
                     BoxSink{&s, nullptr, (long long)k * a.plane, a.nx});
            }
            if (gwp && act) {
                gwp[3 * i] = gx;
                gwp[3 * i + 1] = gy;
                gwp[3 * i + 2] = gzw;
            }
#pragma unroll
            for (int q = 0; q < kTrajProfiles; ++q) accs[q] = q == pi ? acc : accs[q];
        }
    }
    if constexpr (BOX != kWindows && SUMS) flush_box(box, s, a.plane, a.nx);
#pragma unroll
    for (int q = 0; q < kTrajProfiles; ++q) {
        if (q >= np) break;
        if (!takes_radius<BOX>(robots[p0 + q].R)) continue;
        float v = accs[q];
        for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
        if (lane == 0) f[(long long)(p0 + q) * a.T + t] = v;
    }
}

}  // namespace

// Boxes take waypoints with four distinct corners; maps one cell wide or tall
// are taken through walks over the map.
int box_kind(const EvalParams& p) { return p.nx > 1 && p.ny > 1 ? (wide_radius(p.R) ? 2 : 1) : 0; }

void mark_zero_taps(EvalParams& p) {
    for (auto& row : p.K)
        for (float& k : row)
            if (!(k > 0.0f)) k = __builtin_nanf("");
}

pct_status launch_zero(float* p, long long n, hipStream_t s) {
    if (!p || n <= 0) return PCT_OK;
    hipLaunchKernelGGL(k_zero, dim3(grid_for(n)), dim3(kBlock), 0, s, p, n);
    PCT_LAUNCH_CHECK();
    return PCT_OK;
}

static SampleArgs make_sample_args(const pct_grid& g, int N, float d_ref, float w_z, int T, int W) {
    SampleArgs a{};
    a.x0 = g.x0;
    a.y0 = g.y0;
    a.res = g.res;
    a.inv_res = (float)(1.0 / (double)g.res);
    a.d_ref = d_ref;
    a.w_z = w_z;
    a.nx = g.nx;
    a.ny = g.ny;
    a.N = N;
    a.plane = (long long)g.nx * g.ny;
    a.T = T;
    a.W = W;
    return a;
}

pct_status launch_sample_fwd(const float* cost, const float* ground, const pct_grid& g, int N, float d_ref, float w_z,
                             const float* wp, const int* slice, int T, int W, float* f, hipStream_t s) {
    const SampleArgs a = make_sample_args(g, N, d_ref, w_z, T, W);
    const int blocks = (T + kBlock / 64 - 1) / (kBlock / 64);
    hipLaunchKernelGGL(k_sample_fwd, dim3(blocks), dim3(kBlock), 0, s, cost, ground, wp, slice, a, f);
    PCT_LAUNCH_CHECK();
    return PCT_OK;
}

pct_status launch_sample_bwd(const float* cost, const float* ground, const float* ceil, const pct_grid& g, int N,
                             float d_ref, float w_z, const float* wp, const int* slice, int T, int W, const float* gf,
                             float* gwp, float* gcost, float* gground, const EvalParams* ep, const int* aG,
                             const int* aC, float* gz, long long n_points, bool fixed, hipStream_t s) {
    const SampleArgs a = make_sample_args(g, N, d_ref, w_z, T, W);
    Sink sk{};
    sk.fixed = fixed;
    sk.gG = gground;
    sk.gC = nullptr;
    sk.aG = aG;
    sk.aC = aC;
    sk.gz = gz;
    sk.n_points = n_points;
    EvalParams p = ep ? *ep : EvalParams{};
    const long long n = (long long)T * W;
    if (n == 0) return PCT_OK;
    const dim3 blocks((unsigned)((n + kBlock - 1) / kBlock));
    if (ep && box_kind(p) != 0) {
        mark_zero_taps(p);
        if (wide_radius(p.R))
            hipLaunchKernelGGL(k_sample_bwd<kWideBoxes>, blocks, dim3(kBlock), 0, s, cost, ground, ceil, wp, slice, a,
                               gf, gwp, gcost, p, sk);
        else
            hipLaunchKernelGGL(k_sample_bwd<kBoxes>, blocks, dim3(kBlock), 0, s, cost, ground, ceil, wp, slice, a, gf, gwp,
                           gcost, p, sk);
    } else if (ep) {
        hipLaunchKernelGGL(k_sample_bwd<kWindows>, blocks, dim3(kBlock), 0, s, cost, ground, ceil, wp, slice, a, gf,
                           gwp, gcost, p, sk);
    } else {
        hipLaunchKernelGGL(k_sample_bwd<kDense>, blocks, dim3(kBlock), 0, s, cost, ground, ceil, wp, slice, a, gf, gwp,
                           gcost, p, sk);
    }
    PCT_LAUNCH_CHECK();
    return PCT_OK;
}

pct_status launch_eval_bwd(const float* ground, const float* ceil, const float* gcost, const EvalParams& p,
                           float* gground, float* gceil, bool fixed, hipStream_t s) {
    Sink sk{};
    sk.fixed = fixed;
    sk.gG = gground;
    sk.gC = gceil;
    // the largest tile whose box fits; radii that fit none walk their windows
    // over the map
    for (const auto& t : {std::make_pair(16, 8), std::make_pair(8, 8), std::make_pair(8, 4), std::make_pair(4, 4)}) {
        if (p.R > kBoxR || !box_fits(t.first + 2 * p.R, t.second + 2 * p.R, p.rp + 1, fixed)) continue;
        EvalParams q = p;
        mark_zero_taps(q);
        const int nbx = (p.nx + 63) / 64, nby = (p.ny + kEvalLook - 1) / kEvalLook;
        const long long work = (long long)nbx * nby * p.N;
        const dim3 blocks((unsigned)std::min<long long>((work + kBlock / 64 - 1) / (kBlock / 64), 4096));
        auto* tiles = fixed ? k_eval_bwd_tiles<true, kTiles> : k_eval_bwd_tiles<false, kTiles>;
        if (wide_radius(p.R)) tiles = fixed ? k_eval_bwd_tiles<true, kWideTiles> : k_eval_bwd_tiles<false, kWideTiles>;
        if (p.R <= kEvalWalkR) tiles = fixed ? k_eval_bwd_tiles<true, kLoneTiles> : k_eval_bwd_tiles<false, kLoneTiles>;
        hipLaunchKernelGGL(tiles, blocks, dim3(kBlock), 0, s, ground, ceil, gcost, q, t.first, t.second, nbx, nby, sk);
        PCT_LAUNCH_CHECK();
        return PCT_OK;
    }
    hipLaunchKernelGGL(k_eval_bwd, dim3(grid_for(p.plane * p.N)), dim3(kBlock), 0, s, ground, ceil, gcost, p, sk);
    PCT_LAUNCH_CHECK();
    return PCT_OK;
}

pct_status launch_route(const float* gG, const float* gC, const int* aG, const int* aC, long long plane, int N,
                        long long n_points, float* gz, bool fixed, hipStream_t s) {
    hipLaunchKernelGGL(k_route, dim3((unsigned)((plane + kBlock - 1) / kBlock)), dim3(kBlock), 0, s, gG, gC, aG, aC,
                       plane, N, n_points, gz, fixed ? 1 : 0);
    PCT_LAUNCH_CHECK();
    return PCT_OK;
}

pct_status launch_fixed_to_float(const int64_t* q, long long n, float* out, hipStream_t s) {
    if (n <= 0) return PCT_OK;
    hipLaunchKernelGGL(k_fixed_to_float, dim3(grid_for(n)), dim3(kBlock), 0, s, (const long long*)q, n, out);
    PCT_LAUNCH_CHECK();
    return PCT_OK;
}

pct_status launch_traj_value_grad(const float* ground, const float* ceil, const int* aG, const int* aC,
                                  const pct_grid& g, int N, const EvalParams* d_robots, int n_profiles, float w_z,
                                  const float* wp, const int* slice, int T, int W, const float* gf, float* f,
                                  float* gwp, float* gground, float* gceil, float* gz, long long n_points,
                                  bool fixed, int kinds, hipStream_t s) {
    const SampleArgs a = make_sample_args(g, N, 0.0f, w_z, T, W);
    Sink sk{};
    sk.fixed = fixed;
    if (gf) {
        sk.gG = gground;
        sk.gC = gceil;
        sk.aG = aG;
        sk.aC = aC;
        sk.gz = n_points > 0 ? gz : nullptr;
        sk.n_points = n_points;
    }
    if ((long long)n_profiles * T == 0) return PCT_OK;
    // profiles per wavefront: as many as leave 16384 wavefronts, four rounds
    // of the chip (64 profiles x 1024 walks on the building: 2.80 ms, at
    // 8192 3.08 ms); one where the windows are walked over the map
    const bool boxes = kinds != 0;
    const int run = boxes ? (int)std::min<long long>(kTrajProfiles, std::max<long long>(1, (long long)n_profiles * T / 16384))
                          : 1;
    const long long waves = (long long)((n_profiles + run - 1) / run) * T;
    const unsigned blocks = (unsigned)((waves + kBlock / 64 - 1) / (kBlock / 64));
    const bool sums = fixed && (sk.gG || sk.gz);
    float* gw = gf ? gwp : nullptr;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kBlock), 0, s, ground, ceil, d_robots, a, n_profiles, run, wp, slice,
                           gf, f, gw, sk);
    };
    if (!boxes) launch(k_traj_value_grad<kWindows, false>);
    if (kinds & 1) {
        if (sums) launch(k_traj_value_grad<kBoxes, true>);
        else launch(k_traj_value_grad<kBoxes, false>);
        PCT_LAUNCH_CHECK();
    }
    if (kinds & 2) {
        if (sums) launch(k_traj_value_grad<kWideBoxes, true>);
        else launch(k_traj_value_grad<kWideBoxes, false>);
    }
    PCT_LAUNCH_CHECK();
    return PCT_OK;
}

}  // namespace pct
