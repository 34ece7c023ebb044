// Path search through the tomogram slices (Sec. III-D) on the GPU.
//
// The graph: nodes are the cells of L layers (chosen slices, normally the
// ones the simplification keeps); a node links to its eight planar
// neighbours on its layer; moving onto node v costs c^N(v) + step length
// (1 or sqrt 2 cells), where c^N is the least c^T over the node and the
// adjacent layers with the same ground elevation, and a node with
// c^N >= c^B cannot be entered; a layer whose ground is equal and whose c^T
// is strictly lower is reached at no cost (a gateway, upwards or downwards).
//
// Instead of a sequential A* the library computes every node's
// shortest-path distance from the start with a parallel label-correcting
// method, then reads a least-cost path back from the distances.  A* with its
// admissible, consistent heuristic ends with the same least cost.
//
// Distances are FP64.  Each edge relaxation is one rounding of
// dist(u) + (c^N(v) + step) (the edge cost itself one rounding of the FP32
// node cost plus the step); rounding is monotone and every cycle contains a
// planar step (gateways only lead to strictly cheaper layers), so every
// order of relaxations ends at the same least fixed point - the least
// rounded path sum - which is also what Dijkstra's algorithm computes.
//
// Tiles of 64 x 64 cells of one layer are the unit of work.  A round
// processes every active tile: one wavefront loads the tile's distances and
// a one-cell halo into LDS, takes what gateways offer from the adjacent
// layers, then sweeps the tile left-to-right, right-to-left, top-to-bottom
// and bottom-to-top (a lane per row or column, each step relaxing the edges
// from the previous column or row) until a full set of sweeps changes
// nothing, or a number of sweeps is done and the tile stays active.  Improved
// cells are written back; a tile whose border cells improved activates its
// planar neighbours, one whose gateway cells improved activates the tile of
// the adjacent layer.  Rounds repeat until no tile is active.
//
// Latency bounds a round: three tiles fit a CU's LDS, each a wavefront whose
// loads and sweep steps wait for one another.  Distance field of the
// six-storey building (30 layers of 1000 x 1000), step by step on one card:
// 23.5 ms; with capped sweeps 18.9 ms, with a visit's loads in two unbroken
// runs 15.6 ms, and with the old distances read again at the end instead of
// held in 128 registers 14.6 ms; since, node costs and first distances in one
// pass and rounds enqueued ahead.  From the first state to the present one,
// timed in turn: 21.6 and 11.9 ms.
#include <limits.h>
#include <math.h>
#include <string.h>

#include "pct_internal.h"
#include "plan_internal.h"

namespace pct {

namespace {

constexpr int kPT = 64;            // tile side, cells
constexpr int kPS = kPT + 1;       // LDS row stride of the distance tile (doubles)
constexpr int kCS = kPT + 1;       // LDS row stride of the node-cost tile (floats)

__device__ __forceinline__ int cidx(int r, int c) { return r * kCS + c; }
// Sweeps of one visit: a round lasts as long as its slowest tile, so a tile
// that is not at its fixed point after this many goes on in the next round
// (with its neighbours' news).  The field above, other steps not yet taken: 4 /
// 6 / 8 / 10 / 12 / any number of sweeps 20.8 / 19.9 / 18.9 / 19.8 / 20.6 /
// 22.5 ms.
// On graphs of at most kFewTiles tiles no other tile waits for a long visit,
// and every round is two launches: any number of sweeps.  Fields of 2 / 8 / 27
// / 48 tiles, capped and not: 189 / 437 / 500 / 497 us and 112 / 470 / 633 /
// 590 us.
constexpr int kMaxSweeps = 8;
constexpr int kFewTiles = 4;
constexpr double kSqrt2 = 1.4142135623730951;   // sqrt(2) rounded to double

// gateway bits of a node (l, cell)
constexpr unsigned kInFromBelow = 1;   // edge (l-1) -> l
constexpr unsigned kInFromAbove = 2;   // edge (l+1) -> l
constexpr unsigned kOutUp = 4;         // edge l -> (l+1)
constexpr unsigned kOutDown = 8;       // edge l -> (l-1)

struct PlanGeom {
    int nx, ny, L;
    int ntx, nty;
    long long plane;
};

// State of the rounds, kept on the device so that the host looks only every
// few rounds.  Round r's compaction reads the slot of round r - 1 (complete),
// fills slot r % 3, which the relaxation goes on to use, and clears the one
// of round r + 1.
struct PlanStatus {
    unsigned n_list;                // tiles asked for this round (kListCap are taken)
    unsigned done;                  // no active tile, or the goal's distance is final
    unsigned long long rest_key;    // least key of the active tiles not taken
    unsigned long long act_key;     // least key of those the round's relaxation activated
    double band, settled;
    long long tiles;                // rounds and tile visits before this round
    int rounds;
};

__device__ __forceinline__ void clear_round(PlanStatus* st) {
    st->n_list = 0u;
    st->rest_key = ~0ull;
    st->act_key = ~0ull;
}

// Tiles of one round: the launches have that many workgroups, those past the
// list's end leave at once; what is beyond waits for the next round (768
// tiles run at a time).
constexpr int kListCap = 2048;
constexpr int kRoundsAhead = 8;   // rounds enqueued between two looks

PlanGeom make_plan_geom(int nx, int ny, int L) {
    PlanGeom g;
    g.nx = nx;
    g.ny = ny;
    g.L = L;
    g.ntx = (nx + kPT - 1) / kPT;
    g.nty = (ny + kPT - 1) / kPT;
    g.plane = (long long)nx * ny;
    return g;
}

// Node cost (+inf where the node cannot be entered), gateway bits and the
// distances' first value (+inf; the start takes 0 on its tile's first visit),
// and an active flag for the start's tile alone.  A lane takes kPrepLayers
// layers of its cell, so that a layer's ground and cost are read 1.25 times
// instead of three (one node per thread: 295 us for the building's 30 layers,
// distances included).
constexpr int kPrepLayers = 8;

__global__ __launch_bounds__(256) void k_plan_prep(const float* __restrict__ cost, const float* __restrict__ ground,
                                                   const int* __restrict__ layers, PlanGeom g, float cB,
                                                   float* __restrict__ cn, uint8_t* __restrict__ gw,
                                                   double* __restrict__ dist, unsigned* __restrict__ flag,
                                                   unsigned long long* __restrict__ key, int n_tiles, int t0,
                                                   double delta, PlanStatus* __restrict__ st) {
    const long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long n_threads = (long long)gridDim.x * blockDim.x;
    if (blockIdx.y == 0) {
        if (c < 3) {
            clear_round(&st[c]);
            st[c].done = 0u;
            st[c].band = delta;
            st[c].settled = INFINITY;
            st[c].tiles = 0;
            st[c].rounds = 0;
            if (c == 2) st[c].act_key = 0ull;   // the start's tile, before round 0
        }
        for (long long i = c; i < n_tiles; i += n_threads) {
            flag[i] = i == t0 ? 1u : 0u;
            key[i] = i == t0 ? 0ull : ~0ull;   // bits of +0.0
        }
    }
    if (c >= g.plane) return;
    const int l0 = (int)blockIdx.y * kPrepLayers;
    float e[kPrepLayers + 2], t[kPrepLayers + 2];   // layers l0 - 1 .. l0 + kPrepLayers
#pragma unroll
    for (int u = 0; u < kPrepLayers + 2; ++u) {
        const long long o = (long long)layers[min(max(l0 - 1 + u, 0), g.L - 1)] * g.plane + c;
        e[u] = ground[o];
        t[u] = cost[o];
    }
#pragma unroll
    for (int u = 1; u <= kPrepLayers; ++u) {
        const int l = l0 - 1 + u;
        if (l >= g.L) break;
        float n = t[u];
        unsigned bits = 0;
        if (l + 1 < g.L && e[u + 1] == e[u]) {
            n = fminf(n, t[u + 1]);
            if (t[u + 1] < t[u]) bits |= kOutUp;
            if (t[u] < t[u + 1]) bits |= kInFromAbove;
        }
        if (l > 0 && e[u - 1] == e[u]) {
            n = fminf(n, t[u - 1]);
            if (t[u - 1] < t[u]) bits |= kOutDown;
            if (t[u] < t[u - 1]) bits |= kInFromBelow;
        }
        const long long i = (long long)l * g.plane + c;
        cn[i] = n < cB ? n : INFINITY;
        gw[i] = (uint8_t)bits;
        dist[i] = INFINITY;
    }
}

// Lane i receives lane i-1's (i+1's) value, the edge lane `edge`.
__device__ __forceinline__ double from_lane_below(double v, double edge) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v), e = __builtin_bit_cast(unsigned long long, edge);
    const int lo = __builtin_amdgcn_update_dpp((int)(unsigned)e, (int)(unsigned)u, 0x138, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(unsigned)(e >> 32), (int)(unsigned)(u >> 32), 0x138, 0xf, 0xf, false);
    return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}
__device__ __forceinline__ double from_lane_above(double v, double edge) {
    const unsigned long long u = __builtin_bit_cast(unsigned long long, v), e = __builtin_bit_cast(unsigned long long, edge);
    const int lo = __builtin_amdgcn_update_dpp((int)(unsigned)e, (int)(unsigned)u, 0x130, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp((int)(unsigned)(e >> 32), (int)(unsigned)(u >> 32), 0x130, 0xf, 0xf, false);
    return __builtin_bit_cast(double, ((unsigned long long)(unsigned)hi << 32) | (unsigned)lo);
}

// Relaxation of one direction over the tile in LDS.  Lane q walks the
// q-th row (horizontal sweeps) or column (vertical sweeps); at each step it
// relaxes the node's three in-edges from the previous step: its own
// previous node and the diagonal ones, which are the neighbour lanes'
// previous nodes (taken from their registers, so the lanes advance in
// lockstep) or, for the edge lanes, halo cells.  A lane touches only its
// own row or column of the tile in LDS during a sweep.
template <bool VERT, bool REV>
__device__ __forceinline__ bool sweep(double* sd, const double (*hz)[kPT + 2], const float* scn, int q) {
    // node (r, c) of the tile is sd[r * kPS + c]; the halo lines (row -1,
    // row 64, column -1, column 64, each indexed from -1 to 64) are in hz,
    // a separate array, so that their loads can run ahead of the stores
    bool changed = false;
    double prev = VERT ? hz[REV ? 1 : 0][q + 1] : hz[REV ? 3 : 2][q + 1];   // halo before the first step
#pragma unroll 8
    for (int i = 0; i < kPT; ++i) {
        const int s = REV ? kPT - 1 - i : i;      // step along the sweep
        const int sp = REV ? s + 1 : s - 1;       // previous step
        double* me = VERT ? &sd[s * kPS + q] : &sd[q * kPS + s];
        const float c = VERT ? scn[cidx(s, q)] : scn[cidx(q, s)];
        // halo nodes beside lanes 0 and 63 at the previous step
        const double h0 = VERT ? hz[2][sp + 1] : hz[0][sp + 1];
        const double h1 = VERT ? hz[3][sp + 1] : hz[1][sp + 1];
        const double old = *me;
        const double a = from_lane_below(prev, h0), b = from_lane_above(prev, h1);
        const double ws = (double)c + 1.0, wd = (double)c + kSqrt2;
        // sums are canonical, so the minima need no NaN quieting (old + 0
        // for that reason); from one step to the next lie a lane move, a sum
        // and two minima
        const double now = fmin(fmin(prev + ws, old + 0.0), fmin(a + wd, b + wd));
        changed |= now < old;
        prev = now;
        *me = now;
    }
    return changed;
}

// Non-negative doubles order like their bit patterns.
__device__ __forceinline__ unsigned long long dbits(double v) { return __builtin_bit_cast(unsigned long long, v); }

__global__ __launch_bounds__(64) void k_plan_relax(PlanGeom g, const float* __restrict__ cn,
                                                   const uint8_t* __restrict__ gw, double* __restrict__ dist,
                                                   const unsigned* __restrict__ list, unsigned* __restrict__ flag,
                                                   unsigned long long* __restrict__ key, long long src,
                                                   int max_sweeps, PlanStatus* __restrict__ st) {
    if (blockIdx.x >= min(st->n_list, (unsigned)kListCap)) return;
    __shared__ double sd[kPT * kPS];
    __shared__ double hz[4][kPT + 2];
    __shared__ float scn[kPT * kCS];
    const int q = threadIdx.x;
    const unsigned item = list[blockIdx.x];
    const int t = (int)(item >> 1), again = (int)(item & 1u);
    const int tpl = g.ntx * g.nty;
    const int l = t / tpl, tt = t - l * tpl;
    const int ty = tt / g.ntx, tx = tt - ty * g.ntx;
    const int x0 = tx * kPT, y0 = ty * kPT;
    const long long lo = (long long)l * g.plane;
    const int x = x0 + q;
    const bool xin = x < g.nx;

    // Everything the tile needs is loaded from clamped addresses (off the
    // grid, +inf and no gateway take the place of what comes back), so that
    // the loads stand in two unbroken runs and their latencies overlap:
    // distances of the tile and its one-cell halo with the node costs, then
    // the gateway bits.
    const int xc = min(x, g.nx - 1);
    const int yb = max(y0 - 1, 0);
    const double* db = dist + lo + (long long)yb * g.nx;
    auto at = [&](int r) -> unsigned {   // row r, column xc, from (yb, 0): below 2^27
        return (unsigned)(min(max(y0 + r, 0), g.ny - 1) - yb) * (unsigned)g.nx + (unsigned)xc;
    };
    double orig[kPT], hv[3];
    double* dst[3];
    bool in[3];
    double top = db[at(-1)], bot = db[at(kPT)];
#pragma unroll
    for (int r = 0; r < kPT; ++r) orig[r] = db[at(r)];
    {
        // halo columns x0 - 1 and x0 + 64 (rows -1 .. 64), and the four
        // corners again in the halo rows: 136 values over the lanes
#pragma unroll
        for (int k = 0; k < 3; ++k) {
            const int idx = q + 64 * k;
            int xx, yy;
            dst[k] = nullptr;
            if (idx < 2 * (kPT + 2)) {
                const int side = idx / (kPT + 2), r = idx - side * (kPT + 2);
                xx = side ? x0 + kPT : x0 - 1;
                yy = y0 - 1 + r;
                dst[k] = &hz[2 + side][r];
            } else if (idx < 2 * (kPT + 2) + 4) {
                const int cidx = idx - 2 * (kPT + 2);   // (row -1 | 64) x (column -1 | 64)
                xx = (cidx & 1) ? x0 + kPT : x0 - 1;
                yy = (cidx & 2) ? y0 + kPT : y0 - 1;
                dst[k] = &hz[(cidx & 2) ? 1 : 0][(cidx & 1) ? kPT + 1 : 0];
            } else {
                xx = -1;
                yy = -1;
            }
            in[k] = dst[k] && xx >= 0 && xx < g.nx && yy >= 0 && yy < g.ny;
            hv[k] = dist[lo + (long long)min(max(yy, 0), g.ny - 1) * g.nx + min(max(xx, 0), g.nx - 1)];
        }
    }
    {
        float c[kPT];
        const float* cb = cn + lo + (long long)yb * g.nx;
#pragma unroll
        for (int r = 0; r < kPT; ++r) c[r] = cb[at(r)];
        hz[0][q + 1] = xin && y0 > 0 ? top : INFINITY;
        hz[1][q + 1] = xin && y0 + kPT < g.ny ? bot : INFINITY;
#pragma unroll
        for (int k = 0; k < 3; ++k)
            if (dst[k]) *dst[k] = in[k] ? hv[k] : INFINITY;
#pragma unroll
        for (int r = 0; r < kPT; ++r) {
            sd[r * kPS + q] = xin && y0 + r < g.ny ? orig[r] : INFINITY;
        }
#pragma unroll
        for (int r = 0; r < kPT; ++r) scn[cidx(r, q)] = xin && y0 + r < g.ny ? c[r] : INFINITY;
    }
    // gateways into a node offer the adjacent layer's distance at no cost
    // (lane q updates only its own column here)
    bool moved = false;                        // some node of the tile can improve
    unsigned long long outup = 0, outdn = 0;   // nodes of column q with a gateway up / down
    {
        unsigned long long below = 0, above = 0;   // ... from below / from above
        {
            unsigned b[kPT];
            const uint8_t* gb = gw + lo + (long long)yb * g.nx;
#pragma unroll
            for (int r = 0; r < kPT; ++r) b[r] = gb[at(r)];
#pragma unroll
            for (int r = 0; r < kPT; ++r) {
                const unsigned v = xin && y0 + r < g.ny ? b[r] : 0u;
                below |= (unsigned long long)((v & kInFromBelow) != 0) << r;
                above |= (unsigned long long)((v & kInFromAbove) != 0) << r;
                outup |= (unsigned long long)((v & kOutUp) != 0) << r;
                outdn |= (unsigned long long)((v & kOutDown) != 0) << r;
            }
        }
        constexpr int CB = 16;
        for (int r0 = 0; r0 < kPT; r0 += CB) {
            const unsigned nb = (unsigned)(below >> r0) & 0xffffu, na = (unsigned)(above >> r0) & 0xffffu;
            if (__ballot((nb | na) != 0u) == 0ull) continue;   // uniform
            double pb[CB], pa[CB];
#pragma unroll
            for (int j = 0; j < CB; ++j) {
                const double* me = db + at(r0 + j);
                pb[j] = *(me - ((nb >> j & 1u) ? g.plane : 0));
                pa[j] = *(me + ((na >> j & 1u) ? g.plane : 0));
            }
#pragma unroll
            for (int j = 0; j < CB; ++j) {
                double d = INFINITY;
                if (nb >> j & 1u) d = pb[j] + 0.0;
                if (na >> j & 1u) d = fmin(d, pa[j] + 0.0);
                double* me = &sd[(r0 + j) * kPS + q];
                if (d < *me) {
                    *me = d;
                    moved = true;
                }
            }
        }
        // the start node enters at distance 0 on the first visit of its tile
        const long long so = src - lo - (long long)y0 * g.nx - x0;   // of this layer: row * nx + column
        if (so >= 0 && so % g.nx == q && so / g.nx < kPT && src < lo + g.plane && q < g.nx - x0) {
            double* me = &sd[(int)(so / g.nx) * kPS + q];
            if (0.0 < *me) {
                *me = 0.0;
                moved = true;
            }
        }
    }
    __syncthreads();

    // The tile was at a fixed point of its own edges after its last visit,
    // and only its halo and gateway inputs can have changed since: unless a
    // gateway or the start lowered a node above, or a halo node lowers a
    // border node, nothing in the tile can change.
    {
        auto relax3 = [&](int r, int c, double straight, double d1, double d2) {
            const float cc = scn[cidx(r, c)];
            const double cand = fmin(straight + ((double)cc + 1.0), fmin(d1, d2) + ((double)cc + kSqrt2));
            return cand < sd[r * kPS + c];
        };
        moved |= relax3(0, q, hz[0][q + 1], hz[0][q], hz[0][q + 2]);                    // top
        moved |= relax3(kPT - 1, q, hz[1][q + 1], hz[1][q], hz[1][q + 2]);              // bottom
        moved |= relax3(q, 0, hz[2][q + 1], hz[2][q], hz[2][q + 2]);                    // left
        moved |= relax3(q, kPT - 1, hz[3][q + 1], hz[3][q], hz[3][q + 2]);              // right
    }
    if (again == 0 && !__ballot(moved)) return;

    // Sweep the directions in turn (left-to-right, right-to-left,
    // top-to-bottom, bottom-to-top), skipping a direction when no node has
    // changed since its last sweep: after a sweep, every edge of its
    // direction holds, so the tile is at its fixed point when all four are
    // clean.
    unsigned dirty = 0xFu;
    int left = max_sweeps;
    for (int d = 0; dirty && left > 0; d = (d + 1) & 3) {
        if (!(dirty & (1u << d))) continue;
        --left;
        bool ch;
        if (d == 0) ch = sweep<false, false>(sd, hz, scn, q);
        else if (d == 1) ch = sweep<false, true>(sd, hz, scn, q);
        else if (d == 2) ch = sweep<true, false>(sd, hz, scn, q);
        else ch = sweep<true, true>(sd, hz, scn, q);
        dirty &= ~(1u << d);
        if (__ballot(ch)) dirty = 0xFu & ~(1u << d);
        __syncthreads();
    }

    // write back the nodes that changed (values only go down); note which
    // neighbours must look again and the least changed distance (their
    // priority)
    bool nb_up = false, nb_dn = false, nb_l = false, nb_r = false;
    bool c_ul = false, c_ur = false, c_dl = false, c_dr = false, g_up = false, g_dn = false;
    double vmin = INFINITY;
    const int w = min(kPT, g.nx - x0), h = min(kPT, g.ny - y0);
    const bool qin = q < w;
    // against the distances as they were (only this wavefront writes the
    // tile's in a round), read again rather than held through the sweeps
    constexpr int WB = 16;
    for (int r0 = 0; r0 < kPT; r0 += WB) {
        double was[WB];
#pragma unroll
        for (int j = 0; j < WB; ++j) was[j] = db[at(r0 + j)];
#pragma unroll
        for (int j = 0; j < WB; ++j) {
            const int r = r0 + j;
            const double nd = sd[r * kPS + q];
            if (qin && r < h && nd < was[j]) {
                dist[lo + (long long)(y0 + r) * g.nx + x] = nd;
                vmin = fmin(vmin, nd);
                nb_up |= r == 0;
                nb_dn |= r == h - 1;
                nb_l |= q == 0;
                nb_r |= q == w - 1;
                c_ul |= r == 0 && q == 0;
                c_ur |= r == 0 && q == w - 1;
                c_dl |= r == h - 1 && q == 0;
                c_dr |= r == h - 1 && q == w - 1;
                g_up |= ((outup >> r) & 1ull) != 0;
                g_dn |= ((outdn >> r) & 1ull) != 0;
            }
        }
    }
    const unsigned long long m_up = __ballot(nb_up), m_dn = __ballot(nb_dn), m_l = __ballot(nb_l),
                             m_r = __ballot(nb_r), m_ul = __ballot(c_ul), m_ur = __ballot(c_ur),
                             m_dl = __ballot(c_dl), m_dr = __ballot(c_dr), m_gu = __ballot(g_up),
                             m_gd = __ballot(g_dn);
    for (int o = 32; o > 0; o >>= 1) vmin = fmin(vmin, __shfl_xor(vmin, o, 64));
    if (q == 0) {
        const unsigned long long kv = dbits(vmin);
        bool any = dirty != 0u;
        auto act = [&](int ll, int yy, int xx) {
            if (ll < 0 || ll >= g.L || yy < 0 || yy >= g.nty || xx < 0 || xx >= g.ntx) return;
            const int tn = (ll * g.nty + yy) * g.ntx + xx;
            atomicMin(&key[tn], kv);
            atomicOr(&flag[tn], 1u);
            any = true;
        };
        if (dirty) {   // cut short: its own sweeps go on in the next round (flag 2: past the entry test)
            atomicMin(&key[t], kv);
            atomicOr(&flag[t], 2u);
        }
        if (m_up) act(l, ty - 1, tx);
        if (m_dn) act(l, ty + 1, tx);
        if (m_l) act(l, ty, tx - 1);
        if (m_r) act(l, ty, tx + 1);
        if (m_ul) act(l, ty - 1, tx - 1);
        if (m_ur) act(l, ty - 1, tx + 1);
        if (m_dl) act(l, ty + 1, tx - 1);
        if (m_dr) act(l, ty + 1, tx + 1);
        if (m_gu) act(l + 1, ty, tx);
        if (m_gd) act(l - 1, ty, tx);
        if (any) atomicMin(&st->act_key, kv);
    }
}

// Active tiles whose key (the least distance that activated them) lies in
// the band -> worklist (2 * tile, + 1 for one that was cut short; flag and
// key cleared); the others stay active.  A band with no tile left moves up to
// the least active key + delta.  The search ends when no tile is active, or,
// with a goal, when the least active key (a lower bound on every label still
// to be lowered) exceeds the goal's label.
__global__ __launch_bounds__(256) void k_plan_compact(unsigned* __restrict__ flag, unsigned long long* __restrict__ key,
                                                      int n_tiles, double delta, const double* __restrict__ goal,
                                                      unsigned* __restrict__ list, const PlanStatus* __restrict__ prev,
                                                      PlanStatus* __restrict__ cur, PlanStatus* __restrict__ next) {
    const unsigned long long least = min(prev->rest_key, prev->act_key);
    bool done = prev->done != 0u || least == ~0ull;
    double band = prev->band, settled = prev->settled;
    const double kmin = __builtin_bit_cast(double, least);
    if (!done && goal && kmin > *goal) {
        done = true;
        settled = kmin;
    }
    if (!done && kmin > band) band = kmin + delta;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        cur->done = done;
        cur->band = band;
        cur->settled = settled;
        cur->rounds = prev->rounds + (prev->n_list > 0u);
        cur->tiles = prev->tiles + min(prev->n_list, (unsigned)kListCap);
        clear_round(next);
    }
    if (done) return;
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    const unsigned fl = t < n_tiles ? flag[t] : 0u;
    const unsigned long long kt = fl != 0u ? key[t] : ~0ull;
    const bool on = fl != 0u && kt <= dbits(band);
    const unsigned long long m = __ballot(on);
    const int lane = threadIdx.x & 63;
    unsigned base = 0;
    if (lane == 0 && m) base = atomicAdd(&cur->n_list, (unsigned)__popcll(m));
    base = __shfl(base, 0, 64);
    const unsigned at = base + (unsigned)__popcll(m & ((1ull << lane) - 1ull));
    if (on && at < (unsigned)kListCap) {
        flag[t] = 0u;
        key[t] = ~0ull;
        list[at] = (unsigned)t << 1 | (fl >> 1);
    } else if (fl != 0u) {
        atomicMin(&cur->rest_key, kt);
    }
}

// One wavefront walks back from the goal: lanes 0..9 test the candidate
// predecessors (gateway from below, gateway from above, the eight planar
// neighbours in row-major order of (dy, dx)); the first that matches is
// taken.  out[0] receives the node count (0: goal unreachable, -1: not a
// distance field, -2: more than max_len nodes); path rows are written goal
// first and reversed at the end.
__global__ __launch_bounds__(64) void k_plan_path(PlanGeom g, const float* __restrict__ cn,
                                                  const uint8_t* __restrict__ gw, const double* __restrict__ dist,
                                                  const int* __restrict__ layers, int sx, int sy, int sl, int gx,
                                                  int gy, int gl, int* __restrict__ path, int max_len,
                                                  int* __restrict__ out) {
    const int lane = threadIdx.x;
    long long v = (long long)gl * g.plane + (long long)gy * g.nx + gx;
    const long long s = (long long)sl * g.plane + (long long)sy * g.nx + sx;
    __shared__ int s_layer[PCT_MAX_SLICES];
    __shared__ int s_row[64][3];
    for (int i = lane; i < g.L; i += 64) s_layer[i] = layers[i];
    __syncthreads();
    int len = 0, status = 0;
    // the current node's distance and cost travel with it: each step loads
    // the candidates' distance, cost and gateway bits in one round and takes
    // the chosen one's by a shuffle, so a step waits on one memory round.
    // Path rows collect in LDS and go out 64 at a time (a store in flight
    // would hold up the next step's loads).
    auto flush = [&](int n_rows) {
        __syncthreads();
        if (lane < n_rows) {
            const int r = len - n_rows + lane;
            path[3 * r] = s_row[lane][0];
            path[3 * r + 1] = s_row[lane][1];
            path[3 * r + 2] = s_row[lane][2];
        }
        __syncthreads();
    };
    double dv = dist[v];
    float cv = cn[v];
    int x = gx, y = gy, l = gl;  // v's coordinates travel with it too (no divisions)
    if (dv < INFINITY) {
        for (;;) {
            if (len >= max_len) {
                status = -2;
                break;
            }
            const long long c = (long long)y * g.nx + x;
            if (lane == 0) {
                s_row[len & 63][0] = x;
                s_row[len & 63][1] = y;
                s_row[len & 63][2] = s_layer[l];
            }
            ++len;
            if ((len & 63) == 0) flush(64);
            if (v == s) break;
            long long u = -1;
            double du = 0.0;
            float cu = 0.0f;
            int ux = x, uy = y, ul = l;
            bool ok = false;
            if (lane < 2) {
                const int m = lane == 0 ? l - 1 : l + 1;
                if (m >= 0 && m < g.L) {
                    const long long uu = (long long)m * g.plane + c;
                    const unsigned bit = lane == 0 ? kOutUp : kOutDown;
                    const uint8_t gb = gw[uu];
                    du = dist[uu];
                    cu = cn[uu];
                    ul = m;
                    if ((gb & bit) && du + 0.0 == dv) {
                        u = uu;
                        ok = true;
                    }
                }
            } else if (lane < 10) {
                const int e = lane - 2;
                const int dy = e < 3 ? -1 : (e < 5 ? 0 : 1);
                const int dx = e < 3 ? e - 1 : (e < 5 ? (e == 3 ? -1 : 1) : e - 6);
                const int x2 = x + dx, y2 = y + dy;
                if (x2 >= 0 && y2 >= 0 && x2 < g.nx && y2 < g.ny && cv < INFINITY) {
                    const long long uu = (long long)l * g.plane + (long long)y2 * g.nx + x2;
                    du = dist[uu];
                    cu = cn[uu];
                    ux = x2;
                    uy = y2;
                    const double wgt = (double)cv + ((dx != 0 && dy != 0) ? kSqrt2 : 1.0);
                    if (du + wgt == dv) {
                        u = uu;
                        ok = true;
                    }
                }
            }
            const unsigned long long m = __ballot(ok);
            if (!m) {
                status = -1;
                break;
            }
            const int first = __ffsll((long long)m) - 1;
            v = __shfl(u, first, 64);
            dv = __shfl(du, first, 64);
            cv = __shfl(cu, first, 64);
            x = __shfl(ux, first, 64);
            y = __shfl(uy, first, 64);
            l = __shfl(ul, first, 64);
        }
    }
    if ((len & 63) != 0) flush(len & 63);
    __syncthreads();
    if (status == 0) {
        // reverse rows: start first
        for (int a = lane; a < len / 2; a += 64) {
            const int b = len - 1 - a;
            for (int k = 0; k < 3; ++k) {
                const int tmp = path[3 * a + k];
                path[3 * a + k] = path[3 * b + k];
                path[3 * b + k] = tmp;
            }
        }
    }
    if (lane == 0) out[0] = status == 0 ? len : status;
}

struct PlanWs {
    float* cn;
    uint8_t* gw;
    unsigned* flag;
    unsigned long long* key;
    unsigned* list;
    PlanStatus* st;
    int* layers;
    int* out;
};

size_t plan_ws_layout(const PlanGeom& g, PlanWs* w, void* base) {
    const long long nn = g.plane * g.L;
    const int nt = g.ntx * g.nty * g.L;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t o = off;
        off = align_up(off + bytes);
        return (char*)base + o;
    };
    PlanWs ws;
    ws.cn = (float*)take(sizeof(float) * (size_t)nn);
    ws.gw = (uint8_t*)take((size_t)nn);
    ws.flag = (unsigned*)take(sizeof(unsigned) * (size_t)nt);
    ws.key = (unsigned long long*)take(sizeof(unsigned long long) * (size_t)nt);
    ws.list = (unsigned*)take(sizeof(unsigned) * (size_t)nt);
    ws.st = (PlanStatus*)take(3 * sizeof(PlanStatus));
    ws.layers = (int*)take(sizeof(int) * (size_t)g.L);
    ws.out = (int*)take(sizeof(int) * 4);
    if (w) *w = ws;
    return off;
}

}  // namespace

size_t plan_ws_bytes(int nx, int ny, int L) { return plan_ws_layout(make_plan_geom(nx, ny, L), nullptr, nullptr); }

pct_status launch_plan(const float* cost, const float* ground, int nx, int ny, const int* h_layers, int L, float cB,
                       int sx, int sy, int sl, double* dist, void* ws_base, int* h_rounds, long long* h_tiles,
                       hipStream_t s, double delta, long long goal, double* h_settled) {
    const PlanGeom g = make_plan_geom(nx, ny, L);
    PlanWs w;
    plan_ws_layout(g, &w, ws_base);
    const int nt = g.ntx * g.nty * L;
    PCT_HIP(hipMemcpyAsync(w.layers, h_layers, sizeof(int) * (size_t)L, hipMemcpyHostToDevice, s));
    const long long src = (long long)sl * g.plane + (long long)sy * nx + sx;
    const int t0 = (sl * g.nty + sy / kPT) * g.ntx + sx / kPT;
    hipLaunchKernelGGL(k_plan_prep, dim3((unsigned)((g.plane + 255) / 256), (unsigned)((L + kPrepLayers - 1) / kPrepLayers)),
                       dim3(256), 0, s, cost, ground, w.layers, g, cB, w.cn, w.gw, dist, w.flag, w.key, nt, t0, delta, w.st);
    PCT_LAUNCH_CHECK();
    // Rounds take the active tiles whose activating distance lies within
    // a band of width delta above the least one (tiles roughly in order of
    // distance, as Dijkstra's algorithm takes nodes); a band with no tile
    // left moves up to the least remaining key.  The device keeps the band,
    // the list and the end of the search, so the host enqueues rounds ahead
    // (rounds after the end do nothing: 5 us each) and looks after 2, then 4,
    // then every 8: with one look per round the distance field of the
    // building took 13.9 ms and a query 2.20 ms, so 12.2 and 1.99 (one card).
    const int blocks = std::min(nt, kListCap);
    PlanStatus hs;
    for (int r = 0, ahead = 2;; ahead = std::min(2 * ahead, kRoundsAhead)) {
        for (int i = 0; i < ahead; ++i, ++r) {
            PlanStatus *prev = &w.st[(r + 2) % 3], *cur = &w.st[r % 3], *next = &w.st[(r + 1) % 3];
            hipLaunchKernelGGL(k_plan_compact, dim3((unsigned)((nt + 255) / 256)), dim3(256), 0, s, w.flag, w.key, nt,
                               delta, goal >= 0 ? dist + goal : nullptr, w.list, prev, cur, next);
            PCT_LAUNCH_CHECK();
            hipLaunchKernelGGL(k_plan_relax, dim3((unsigned)blocks), dim3(64), 0, s, g, w.cn, w.gw, dist, w.list, w.flag,
                               w.key, src, nt <= kFewTiles ? INT_MAX : kMaxSweeps, cur);
            PCT_LAUNCH_CHECK();
        }
        PCT_HIP(hipMemcpyAsync(&hs, &w.st[(r + 2) % 3], sizeof hs, hipMemcpyDeviceToHost, s));
        PCT_HIP(hipStreamSynchronize(s));
        if (hs.done) break;
    }
    if (h_rounds) *h_rounds = hs.rounds;
    if (h_tiles) *h_tiles = hs.tiles;
    if (h_settled) *h_settled = hs.settled;
    return PCT_OK;
}

pct_status launch_plan_path(const double* dist, int nx, int ny, int L, int sx, int sy, int sl, int gx, int gy, int gl,
                            int* path, int max_len, void* ws_base, int* h_len, hipStream_t s) {
    const PlanGeom g = make_plan_geom(nx, ny, L);
    PlanWs w;
    plan_ws_layout(g, &w, ws_base);
    hipLaunchKernelGGL(k_plan_path, dim3(1), dim3(64), 0, s, g, w.cn, w.gw, dist, w.layers, sx, sy, sl, gx, gy, gl,
                       path, max_len, w.out);
    PCT_LAUNCH_CHECK();
    int out = 0;
    PCT_HIP(hipMemcpyAsync(&out, w.out, sizeof(int), hipMemcpyDeviceToHost, s));
    PCT_HIP(hipStreamSynchronize(s));
    *h_len = out;
    return PCT_OK;
}

}  // namespace pct
