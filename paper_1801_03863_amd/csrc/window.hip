// window.hip -- D2Q9, one lattice, up to K steps per launch in on-chip
// windows: the path of small and medium lattices, for every collision rule
// and storage form.
//
// A single-step launch of a small lattice costs about 4 us whatever the
// lattice holds: most of the chip idles while a few waves wait for their
// loads, run one collision and store.  Here a block owns a tile of tw x th
// nodes and takes n steps in one launch.  Its window is the tile and the
// n - 1 nodes around it (cut at lattice ends that do not wrap).  The first
// step computes every window node straight from the other buffer, exactly as
// a single-step launch does, and leaves the post-collision populations in LDS
// in their storage form; step s then recomputes the nodes still n - 1 - s
// away from the tile, and the last step writes the tile to HBM.  An axis the
// tile covers whole has no window beyond it: its ends wrap or clamp inside
// LDS.  Every node is computed with the same arithmetic and rounded to the
// storage type after every step, so results are bitwise equal to single
// steps.
//
// One thread computes one node per step.  The window is kept once: a step
// reads it, waits, and writes it back, which costs a second barrier but halves
// the LDS of two buffers, so that an FP64 window of 910 nodes fits the
// 64 KiB every kernel may use.  What bounds it is the latency of one
// collision (a dependent chain of FP64 operations, reciprocals and the 4 x 4
// solve: 1950 cycles in FP64, 1000 for SRT) and, with more than one wave per
// SIMD, VALU issue (1550 cycles a wave); about 2.1 us of a launch lie outside the
// kernel and 1.5 us are its mapping and first loads.  The tile is chosen for
// that (d2q9_window_best).  Measured, us per step, FP64 cavities, one step per
// launch -> windows: 32^2 4.4 -> 1.5, 128^2 4.6 -> 1.8, 257^2 6.2 -> 3.4, 480^2 9.7 ->
// 6.3, 512^2 10.8 -> 7.5; SRT tubes 33 x 27 4.0 -> 1.0, 129 x 123 4.1 -> 1.4.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <stdint.h>

#include "device.hpp"
#include "kernels.hpp"

namespace lbm {

// What the kernel reads, packed into a few lines of kernel arguments: a launch
// of a small lattice is short enough that fetching them counts.
struct WinArgs {
    const void *src;
    void *dst;
    DevStatus *status;
    const int64_t *step_base;
    int64_t step, plane;
    int32_t nx, ny, pitch, bc;
    int32_t tw, th, cap, steps;
    float scale, iscale;
    double omega, omega2, rho0;
    double lid[9];
};

// Rows or columns [lo, hi) a step d steps before the last must compute along
// one axis of n nodes, for a tile [t0, t1): the tile and d nodes around it.
__device__ __forceinline__ void win_range(int t0, int t1, int n, bool whole, bool wrap, int d, int &lo, int &hi)
{
    lo = whole ? 0 : (wrap ? t0 - d : max(0, t0 - d));
    hi = whole ? n : (wrap ? t1 + d : min(n, t1 + d));
}

// Neighbour coordinates of g along an axis inside the window: one node on,
// wrapped or clamped only where the lattice ends inside the window.
__device__ __forceinline__ void win_neighbours(int g, int n, bool whole, bool wrap, int &m, int &p)
{
    m = g - 1;
    p = g + 1;
    if (wrap) {
        if (whole) {
            if (m < 0) m = n - 1;
            if (p >= n) p = 0;
        }
    } else {
        m = max(m, 0);
        p = min(p, n - 1);
    }
}

// Lattice coordinate of a window coordinate on an axis that wraps.
__device__ __forceinline__ int win_wrap(int g, int n)
{
    if (g < 0) g += n;
    if (g >= n) g -= n;
    if ((unsigned)g >= (unsigned)n) g = ((g % n) + n) % n;  // a window longer than the axis
    return g;
}

template <int ST, int CO>
__global__ __launch_bounds__(1024) void k_d2q9_win(WinArgs a)
{
    using C = typename Form<ST>::C;
    using T = typename Form<ST>::T;
    extern __shared__ __align__(16) unsigned char win_lds[];
    T *L = (T *)win_lds;  // nine planes of `cap` nodes, window nodes row-major
    const int cap = a.cap;
    const int nx = a.nx, ny = a.ny;
    const bool xw = a.bc == BC_PERIODIC;
    const bool yw = a.bc == BC_PERIODIC || a.bc == BC_TUBE;
    const bool wholex = gridDim.x == 1, wholey = gridDim.y == 1;
    const int x0 = (int)blockIdx.x * a.tw, y0 = (int)blockIdx.y * a.th;
    const int x1 = min(nx, x0 + a.tw), y1 = min(ny, y0 + a.th);
    const int n = a.steps;
    Inst in;  // what the collision reads
    in.omega = a.omega;
    in.omega2 = a.omega2;
#pragma unroll
    for (int q = 0; q < 9; ++q) in.lid[q] = a.lid[q];
    C ref[9];
    ref9<C>(C(a.rho0), ref);

    // Thread -> window node: the tile's nodes first, row by row, then the
    // rings around it outwards (a ring is what a range of d steps has beyond
    // that of d - 1: up to one row and one column on each side).  The nodes
    // that later steps drop are thus the last threads', and waves drop whole.
    const int tw = x1 - x0, tile = tw * (y1 - y0);
    int i = (int)threadIdx.x, ring = i < tile ? 0 : -1;  // ring < 0: no node
    int left = i - tile;                                 // index beyond the rings passed
    int xl = x0, xh = x1, yl = y0, yh = y1;              // uniform: the range of d steps
    for (int d = 1; d < n; ++d) {
        const int px = xh - xl, py = yh - yl;
        win_range(x0, x1, nx, wholex, xw, d, xl, xh);
        win_range(y0, y1, ny, wholey, yw, d, yl, yh);
        const int m = (xh - xl) * (yh - yl) - px * py;
        if (ring < 0) {
            if (left < m) {
                ring = d;
                i = left;
            }
            left -= m;
        }
    }
    // xl .. yh is now the window.  Quotients of indices below 1024 by a float
    // estimate, exact after one correction.
    int x, y;
    if (ring <= 0) {
        y = (int)((float)i * __builtin_amdgcn_rcpf((float)tw));
        x = i - y * tw;
        if (x < 0) { --y; x += tw; }
        if (x >= tw) { ++y; x -= tw; }
        x += x0;
        y += y0;
    } else {
        int oxl, oxh, oyl, oyh, ixl, ixh, iyl, iyh;  // the ring's outer and inner range
        win_range(x0, x1, nx, wholex, xw, ring, oxl, oxh);
        win_range(y0, y1, ny, wholey, yw, ring, oyl, oyh);
        win_range(x0, x1, nx, wholex, xw, ring - 1, ixl, ixh);
        win_range(y0, y1, ny, wholey, yw, ring - 1, iyl, iyh);
        const int w = oxh - oxl, h = iyh - iyl, rows = ((iyl - oyl) + (oyh - iyh)) * w;
        const bool row = i < rows;
        const int k = row ? i : i - rows, len = row ? w : h;
        const bool second = k >= len;
        const int o = second ? k - len : k;
        x = row ? oxl + o : (second || oxl == ixl ? oxh - 1 : oxl);
        y = row ? (second || oyl == iyl ? oyh - 1 : oyl) : iyl + o;
    }
    // LDS addresses of the node and of the nine slots it pulls from, and its
    // role, hold for every step.
    const int ww = xh - xl;
    const bool own = ring == 0;
    const int last = ring < 0 ? -1 : n - 1 - ring;  // last step that computes the node
    int wr = 0, rd[9];
    {
        int xm, xp, ym, yp;
        win_neighbours(x, nx, wholex, xw, xm, xp);
        win_neighbours(y, ny, wholey, yw, ym, yp);
        const int cc = x - xl, cm = xm - xl, cp = xp - xl;
        const int rc = (y - yl) * ww, rm = (ym - yl) * ww, rp = (yp - yl) * ww;
        const int o[9] = {rc + cc, rc + cm, rm + cc, rc + cp, rp + cc, rm + cm, rm + cp, rp + cp, rp + cm};
        wr = o[0];
#pragma unroll
        for (int q = 0; q < 9; ++q) rd[q] = q * cap + o[q];
    }
    const int role = role9(x, y, nx, ny, a.bc);  // never depends on a wrapped coordinate

    int bad_step = -1, guarded = 0;
    T sv[9];
    // One step of this thread's node from its pulled populations.
    auto collide = [&](C (&f)[9], int s) {
        const int fl = node9<ST, CO>(f, role, in);
        if (own) {
            if ((fl & 1) && bad_step < 0) bad_step = s;
            guarded += (fl >> 1) & 1;
        }
#pragma unroll
        for (int q = 0; q < 9; ++q) sv[q] = to_storage<ST>(f[q], ref[q], a.scale);
    };
    if (last >= 0) {
        const int lx = xw ? win_wrap(x, nx) : x, ly = yw ? win_wrap(y, ny) : y;
        C f[9];
        pull9<ST>((const T *)a.src, a.plane, lx, ly, a.pitch, neighbours(lx, ly, nx, ny, a.bc), ref, a.iscale, f);
        collide(f, 0);
    }
    for (int s = 1; s < n; ++s) {
        if (s > 1) lds_barrier();  // every read of the last step before the writes
        if (last >= s - 1) {
            T *p = L + wr;
#pragma unroll
            for (int q = 0; q < 9; ++q) p[q * cap] = sv[q];
        }
        lds_barrier();
        if (last >= s) {
            C f[9];
#pragma unroll
            for (int q = 0; q < 9; ++q) f[q] = load<ST>(L + rd[q], ref[q], a.iscale);
            collide(f, s);
        }
    }
    if (own) {
        char *b = (char *)a.dst + plane_bytes(x, y, a.pitch, (int)sizeof(T));
        const int64_t PB = a.plane * (int64_t)sizeof(T);
#pragma unroll
        for (int q = 0; q < 9; ++q) *(T *)(b + q * PB) = sv[q];
    }
    // Status: rare events.  The smallest (step, node) of the wave, and one
    // addition per lane that kept start points.
    if (__ballot(bad_step >= 0 || guarded != 0) != 0ull) {
        const int64_t s0 = a.step + (a.step_base ? *a.step_base : 0);
        report_key(a.status, bad_step >= 0 ? event_key(s0 + bad_step, y * nx + x) : ~0ull);
        if (guarded != 0) {
            atomicOr(&a.status->flags, 2u);
            atomicAdd((unsigned long long *)&a.status->guarded, (unsigned long long)guarded);
        }
    }
}

// --------------------------------------------------------------------------
// Host side
// --------------------------------------------------------------------------

namespace {

size_t elem_of(int st) { return st == ST_F64 ? 8 : (st == ST_F16DEV ? 2 : 4); }

template <int ST>
hipError_t win_go(int coll, const WinArgs &w, dim3 grid, int threads, hipStream_t s)
{
    const size_t smem = 9 * (size_t)w.cap * sizeof(typename Form<ST>::T);
    switch (coll) {
    case CO_MINXENT4: hipLaunchKernelGGL((k_d2q9_win<ST, CO_MINXENT4>), grid, dim3(threads), smem, s, w); break;
    case CO_MINXENT2: hipLaunchKernelGGL((k_d2q9_win<ST, CO_MINXENT2>), grid, dim3(threads), smem, s, w); break;
    case CO_SRT: hipLaunchKernelGGL((k_d2q9_win<ST, CO_SRT>), grid, dim3(threads), smem, s, w); break;
    case CO_TRT: hipLaunchKernelGGL((k_d2q9_win<ST, CO_TRT>), grid, dim3(threads), smem, s, w); break;
    case CO_MRT: hipLaunchKernelGGL((k_d2q9_win<ST, CO_MRT>), grid, dim3(threads), smem, s, w); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Widest range along an axis d steps before the last (as win_range, for the
// largest tile).
int win_extent(int t, int n, bool whole, bool wrap, int d)
{
    if (whole) return n;
    return wrap ? t + 2 * d : std::min(n, t + 2 * d);
}

}  // namespace

int d2q9_window_cap(int st) { return (int)std::min<size_t>(1024, 65536 / (9 * elem_of(st))); }

int d2q9_window_best(int st, int coll, int nx, int ny, int bc, const int *ks, int nk, double below, WindowTile *out,
                     double *us_per_step)
{
    // Time of a launch in us: a fixed part (launch, mapping, first loads), the
    // lattice's bytes at the rate of launches whose state the caches hold, and
    // per step the exchange through LDS and the issue of the waves that share
    // a SIMD; the blocks of a compute unit that its LDS (160 KiB) or registers do
    // not hold at once come one after another.  Fitted to 4,500 launches of 4 to
    // 64 steps (12^2 to 1600^2, every rule and form): off by 7-15% rms, by 15-28%
    // before the blocks in turn were counted.
    const bool newton = coll == CO_MINXENT4 || coll == CO_MINXENT2;
    const double issue_of[2][4] = {{0.66, 0.64, 0.39, 0.41}, {0.95, 0.89, 0.64, 0.66}};
    const double issue = issue_of[newton][st], exchange = 0.3;
    const double fixed = 5.3 + (double)nx * ny * 18 * elem_of(st) / 18e6;
    const int simd_waves = newton && (st == ST_F64 || st == ST_F32N64) ? 4 : (newton || st == ST_F64 ? 7 : 8);
    const int cap = d2q9_window_cap(st);
    const bool xw = bc == BC_PERIODIC, yw = bc == BC_PERIODIC || bc == BC_TUBE;
    // Grids of tiles: for each width, the fewest rows that give each compute unit
    // r blocks.
    struct Grid {
        WindowTile t;
        int blocks, waves;  // of a compute unit; of a tile
    } grids[16 * 6];
    int n = 0;
    for (const int tw0 : {nx, 4, 6, 8, 10, 12, 14, 16, 18, 20, 24, 28, 32, 40, 48, 64}) {
        if (tw0 > nx) break;
        const int gx = (nx + tw0 - 1) / tw0, tw = (nx + gx - 1) / gx;
        if (tw > cap || (n && grids[n - 1].t.tw == tw)) continue;
        for (int r = 1, last = 0; r <= 6; ++r) {
            const int gy0 = std::max(1, std::min(ny, kWindowCus * r / gx));
            const int th = (ny + gy0 - 1) / gy0, gy = (ny + th - 1) / th;
            if (gy == last) continue;
            last = gy;
            if ((int64_t)tw * th > cap) continue;
            const int blocks = (int)(((int64_t)gx * gy + kWindowCus - 1) / kWindowCus);
            grids[n++] = Grid{WindowTile{tw, th, gx, gy}, blocks, (tw * th + 63) / 64};
        }
    }
    // The no-allocation call plans on every call, so a grid is left as soon as its
    // steps cannot be cheap enough, without its windows at first (the choice of a
    // starting shape, us of host time with every grid summed up / so: 17^2 15 / 1.8,
    // 128^2 11 / 3.4, 257^2 13 / 3.8, 1000^2 5.5 / 1.7).
    int found = -1;
    for (int i = 0; i < nk; ++i) {
        const int k = ks[i];
        double best = below * k;
        for (const Grid *g = grids; g < grids + n; ++g) {
            const int tw = g->t.tw, th = g->t.th;
            const bool wx = g->t.gx == 1, wy = g->t.gy == 1;
            const double work = issue * g->blocks * g->waves / 4.0;
            if (fixed + k * (exchange + std::max(issue, work)) * (1 - 1e-9) >= best) continue;
            const int64_t m0 = (int64_t)win_extent(tw, nx, wx, xw, k - 1) * win_extent(th, ny, wy, yw, k - 1);
            if (m0 > cap) continue;
            const int resident = std::max(1, std::min((int)(163840 / (9 * elem_of(st) * m0)),
                                                      4 * simd_waves / (int)((m0 + 63) / 64)));
            const int turns = (g->blocks + resident - 1) / resident;
            if (fixed + k * (turns * exchange + std::max(turns * issue, work)) * (1 - 1e-9) >= best) continue;
            double c = fixed;
            for (int left = g->blocks; left > 0 && c < best; left -= resident) {
                const int blocks = std::min(left, resident);
                for (int d = k - 1; d >= 0 && c < best; --d) {
                    const int m = win_extent(tw, nx, wx, xw, d) * win_extent(th, ny, wy, yw, d);
                    c += exchange + issue * std::max(1.0, blocks * ((m + 63) / 64) / 4.0);
                }
            }
            if (c < best) {
                best = c;
                found = i;
                *out = g->t;
            }
        }
        below = std::min(below, best / k);
    }
    if (us_per_step && found >= 0) *us_per_step = below;
    return found;
}

hipError_t launch_d2q9_window(int st, int coll, const void *src, void *dst, const StepArgs &a, hipStream_t s)
{
    const bool xw = a.bc == BC_PERIODIC, yw = a.bc == BC_PERIODIC || a.bc == BC_TUBE;
    const WindowTile &t = a.win;
    const Inst &in = a.one;
    if (a.max_steps < 1 || t.tw < 1 || t.th < 1 || t.gx < 1 || t.gy < 1 || t.gy > 65535) return hipErrorInvalidValue;
    const int64_t n = (int64_t)win_extent(t.tw, in.nx, t.gx == 1, xw, a.max_steps - 1) *
                      win_extent(t.th, in.ny, t.gy == 1, yw, a.max_steps - 1);
    if (n > d2q9_window_cap(st) || (int64_t)t.tw * t.gx < in.nx || (int64_t)t.th * t.gy < in.ny)
        return hipErrorInvalidValue;
    WinArgs w{};
    w.src = src;
    w.dst = dst;
    w.status = a.status;
    w.step_base = a.step_base;
    w.step = a.step;
    w.plane = in.plane;
    w.nx = in.nx;
    w.ny = in.ny;
    w.pitch = in.pitch;
    w.bc = a.bc;
    w.tw = t.tw;
    w.th = t.th;
    w.cap = (int32_t)n;
    w.steps = a.max_steps;
    w.scale = a.fp16_scale;
    w.iscale = a.fp16_iscale;
    w.omega = in.omega;
    w.omega2 = in.omega2;
    w.rho0 = in.rho0;
    std::copy(in.lid, in.lid + 9, w.lid);
    const dim3 grid(t.gx, t.gy);
    const int threads = (int)((n + 63) / 64 * 64);
    switch (st) {
    case ST_F64: return win_go<ST_F64>(coll, w, grid, threads, s);
    case ST_F32N64: return win_go<ST_F32N64>(coll, w, grid, threads, s);
    case ST_F32: return win_go<ST_F32>(coll, w, grid, threads, s);
    case ST_F16DEV: return win_go<ST_F16DEV>(coll, w, grid, threads, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace lbm
