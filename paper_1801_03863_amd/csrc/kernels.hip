// kernels.hip -- fused stream-and-collide kernels of MinxEnt-LBM for gfx950.
//
// One thread owns one node per row it visits.  Each time step it pulls the
// nine (or three) populations that stream into its node from the previous
// post-collision state (Sec. II.A: f_a(x + v_a, t+1) = post-collision f_a(x, t),
// read here as f_a(x) <- f*_a(x - v_a)), applies the node's role -- the
// collision rule on fluid nodes, full-way bounce-back on walls, the
// equilibrium of the lid's density and velocity on the lid (Sec. IV.E) -- and
// writes its nine post-collision populations to the other buffer.
//
// Layout: structure of arrays, one plane per direction of ny rows of nx
// values, x fastest, each row starting a 128-byte line (rows `pitch`
// elements apart, nx rounded up to whole lines; the padding is never read),
// so every plane read is a unit-stride row shifted by at most one element and
// every write is aligned and unit-stride.  Planes follow each other at a
// stride of ny * pitch rounded up to 64 elements, plus, for a
// large single lattice, a tuned pad that is a multiple of 256 bytes, so every
// plane starts 256-byte aligned.  The single-step kernels read and write
// every population exactly once per step; they are bound by HBM bandwidth in
// the FP64, FP32 and FP32-storage/FP64-compute forms, and by VALU issue (the
// logarithms, reciprocals and 4 x 4 solve of the Newton step) when the
// populations are FP16 deviations.  The kernels that take several steps per
// launch read and write every population once per launch, and HBM then no longer
// bounds the MinxEnt rules: two D2Q9 steps with the rows between in LDS, or a
// batch's small lattices whole in LDS (further down); up to 64 in windows in LDS
// (window.hip); two to four with the rows between in registers (pipeline.hpp); up
// to 32 D1Q3 steps with the nodes in registers (tube.hip).
//
// Slots of boundary nodes whose upstream node lies outside the lattice read a
// clamped (in-bounds) location; their values are bounced outward and never
// reach a fluid node.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <stdint.h>

#include "device.hpp"
#include "kernels.hpp"

namespace lbm {

// --------------------------------------------------------------------------
// D2Q9, one lattice.  Block = BX x BY threads (BX a multiple of 64, so a wave
// never spans two rows); it covers BX columns and BY*RPT rows.
// --------------------------------------------------------------------------

// WPE > 0 asks the compiler for at least WPE waves per SIMD (a register
// budget of 512/WPE VGPRs), trading registers for occupancy.
template <int ST, int CO, int BX, int BY, int RPT, int NT = 0, int WPE = 0>
__global__ __launch_bounds__(BX *BY) __attribute__((amdgpu_waves_per_eu(WPE > 0 ? WPE : 1)))
void k_d2q9(const typename Form<ST>::T *__restrict__ src, typename Form<ST>::T *__restrict__ dst, StepArgs a)
{
    using C = typename Form<ST>::C;
    // NT bit 3: the wave runs at raised issue priority until its loads are
    // in flight, so a new wave gets its memory requests out ahead of the
    // arithmetic of older waves.
    if constexpr ((NT & 8) != 0) __builtin_amdgcn_s_setprio(2);
    const Inst &in = a.one;
    const int nx = in.nx, ny = in.ny, pitch = in.pitch;
    const int64_t P = in.plane;
    int tx, ty;
    tile_of_block(a.xcd_swizzle, a.tiles_x, tx, ty);
    const int x = tx * BX + (int)threadIdx.x;
    const bool xin = x < nx;
    const int xs = xin ? x : nx - 1;
    const Cols cols = columns(xs, tx == 0 || tx == a.tiles_x - 1, nx, a.bc, sizeof(typename Form<ST>::T));
    C ref[9];
    ref9<C>(C(in.rho0), ref);
    int bad = kNoNode;
    int guarded = 0;
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        // A wave never spans two rows (BX is a multiple of 64), so y is
        // wave-uniform; saying so keeps all row logic in scalar registers.
        const int y = __builtin_amdgcn_readfirstlane((ty * RPT + k) * BY + (int)threadIdx.y);
        if (y >= ny) break;
        if (a.bc == BC_CAVITY && y == ny - 1) {
            if (xin) push_lid<ST, (NT & 2) != 0>(dst, P, x, y, pitch, in, ref, a.fp16_scale);
            continue;
        }
        const Nb n = neighbours(0, y, 1, ny, a.bc);  // rows only
        C f[9];
        {
            typename Form<ST>::T raw[9];
            pull9_cols<ST, nl_mode(NT)>(src, P, y, n.ym, n.yp, pitch, cols.cc, cols.cm, cols.cp, raw);
            if constexpr ((NT & 8) != 0) __builtin_amdgcn_s_setprio(0);
#pragma unroll
            for (int q = 0; q < 9; ++q) f[q] = load<ST>(&raw[q], ref[q], a.fp16_iscale);
        }
        const int fl = node9_row<ST, CO>(f, xs, y, nx, ny, a.bc, in);
        if (xin && (fl & 1)) bad = min(bad, y * nx + x);
        guarded += __popcll(__ballot(xin && (fl & 2)));
        if (xin) push9_xy<ST, (NT & 2) != 0>(dst, P, x, y, pitch, f, ref, a.fp16_scale);
    }
    report(a.status, bad, guarded, a.step, a.step_base);
}

// LDS-staged form.  A block of BX threads covers BX columns of RY rows, one
// row at a time.  For each of the nine planes it stages the source row
// window [x0 - 1, x0 + BX] that the row's nodes pull from (row shifted by the
// plane's vertical velocity, columns by at most one) in LDS: the aligned
// BX-wide middle with 16-byte vector loads when every row start is 16-byte
// aligned (the row pitch a multiple of the vector width), element by element otherwise,
// and the two edge columns by single loads.  Window columns outside the
// lattice hold the wrap/clamp source of the edge nodes, so every node reads
// exactly what the direct forms read and results are bitwise equal.
template <int ST, int CO, int BX, int RY, int NT = 0>
__global__ __launch_bounds__(BX) void k_d2q9_stage(const typename Form<ST>::T *__restrict__ src,
                                                   typename Form<ST>::T *__restrict__ dst, StepArgs a)
{
    using C = typename Form<ST>::C;
    using T = typename Form<ST>::T;
    constexpr int V = 16 / sizeof(T);  // elements per vector
    // LDS row: [V-1] left edge, [V, V+BX) middle (16-byte aligned), [V+BX]
    // right edge; the row stride is a multiple of 16 bytes.
    constexpr int W = BX + 2 * V;
    __shared__ __align__(16) T win[9][W];
    const Inst &in = a.one;
    const int nx = in.nx, ny = in.ny, pitch = in.pitch;
    const int64_t P = in.plane;
    const bool xw = a.bc == BC_PERIODIC;
    int tx, ty;
    tile_of_block(a.xcd_swizzle, a.tiles_x, tx, ty);
    const int t = (int)threadIdx.x;
    const int x0 = tx * BX;
    const int x = x0 + t;
    const bool xin = x < nx;
    const int xs = xin ? x : nx - 1;
    const bool vec = (pitch % V) == 0;
    C ref[9];
    ref9<C>(C(in.rho0), ref);
    int bad = kNoNode;
    int guarded = 0;
    for (int r = 0; r < RY; ++r) {
        const int y = ty * RY + r;  // uniform across the block
        if (y >= ny) break;
        if (a.bc == BC_CAVITY && y == ny - 1) {
            if (xin) push_lid<ST, (NT & 2) != 0>(dst, P, x, y, pitch, in, ref, a.fp16_scale);
            continue;
        }
        const Nb n = neighbours(0, y, 1, ny, a.bc);  // rows only
        // Stage the nine windows.
        for (int i = t; i < 9 * (BX / V); i += BX) {
            const int q = i / (BX / V), k = i - q * (BX / V);
            const int vy = cy9(q);
            const int ys = vy > 0 ? n.ym : (vy < 0 ? n.yp : y);
            const T *row = src + (int64_t)q * P + (int64_t)ys * pitch;
            const int c0 = x0 + k * V;
            if (vec && c0 + V <= nx) {
                const u32x4 *p = (const u32x4 *)(row + c0);
                u32x4 w;
                if constexpr ((NT & 1) != 0) w = __builtin_nontemporal_load(p);
                else w = *p;
                *(u32x4 *)&win[q][V + k * V] = w;
            } else {
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    const int c = c0 + e;
                    const int ce = c < nx ? c : ((c == nx && xw) ? 0 : nx - 1);
                    win[q][V + k * V + e] = ldraw<T, (NT & 1) != 0>(row + ce);
                }
            }
        }
        if (t < 18) {
            const int q = t >> 1;
            const int vy = cy9(q);
            const int ys = vy > 0 ? n.ym : (vy < 0 ? n.yp : y);
            const int c = (t & 1) ? x0 + BX : x0 - 1;
            const int ce = c < 0 ? (xw ? nx - 1 : 0) : (c >= nx ? ((c == nx && xw) ? 0 : nx - 1) : c);
            win[q][(t & 1) ? V + BX : V - 1] =
                ldraw<T, (NT & 1) != 0>(src + (int64_t)q * P + (int64_t)ys * pitch + ce);
        }
        __syncthreads();
        C f[9];
#pragma unroll
        for (int q = 0; q < 9; ++q) f[q] = load<ST>(&win[q][t + V - cx9(q)], ref[q], a.fp16_iscale);
        __syncthreads();  // the windows are restaged for the next row
        const int fl = node9_row<ST, CO>(f, xs, y, nx, ny, a.bc, in);
        if (xin && (fl & 1)) bad = min(bad, y * nx + x);
        guarded += __popcll(__ballot(xin && (fl & 2)));
        if (xin) push9_xy<ST, (NT & 2) != 0>(dst, P, x, y, pitch, f, ref, a.fp16_scale);
    }
    report(a.status, bad, guarded, a.step, a.step_base);
}

// Software-pipelined form: a block of BX threads walks RPT consecutive rows;
// each thread issues the raw loads of its next row before computing the
// current one, so nine loads per thread are always in flight while the VALU
// works.  Same per-node arithmetic as k_d2q9 (bitwise identical results).
template <int ST, int CO, int BX, int RPT, int NT = 0, int WPE = 0>
__global__ __launch_bounds__(BX) __attribute__((amdgpu_waves_per_eu(WPE > 0 ? WPE : 1))) void k_d2q9_pf(const typename Form<ST>::T *__restrict__ src,
                                                typename Form<ST>::T *__restrict__ dst, StepArgs a)
{
    using C = typename Form<ST>::C;
    using T = typename Form<ST>::T;
    const Inst &in = a.one;
    const int nx = in.nx, ny = in.ny, pitch = in.pitch;
    const int64_t P = in.plane;
    int tx, ty;
    tile_of_block(a.xcd_swizzle, a.tiles_x, tx, ty);
    const int x = tx * BX + (int)threadIdx.x;
    const bool xin = x < nx;
    const int xs = xin ? x : nx - 1;
    const int y0 = ty * RPT;
    const Cols cols = columns(xs, tx == 0 || tx == a.tiles_x - 1, nx, a.bc, sizeof(T));
    C ref[9];
    ref9<C>(C(in.rho0), ref);
    int bad = kNoNode;
    int guarded = 0;
    T raw[9];
    {
        const Nb n = neighbours(0, y0, 1, ny, a.bc);  // rows only
        pull9_cols<ST, nl_mode(NT)>(src, P, y0, n.ym, n.yp, pitch, cols.cc, cols.cm, cols.cp, raw);
    }
#pragma unroll
    for (int k = 0; k < RPT; ++k) {
        const int y = y0 + k;
        if (y >= ny) break;  // uniform across the block
        C f[9];
#pragma unroll
        for (int q = 0; q < 9; ++q) f[q] = load<ST>(&raw[q], ref[q], a.fp16_iscale);
        if (k + 1 < RPT && y + 1 < ny) {
            const Nb n = neighbours(0, y + 1, 1, ny, a.bc);  // rows only
            pull9_cols<ST, nl_mode(NT)>(src, P, y + 1, n.ym, n.yp, pitch, cols.cc, cols.cm, cols.cp, raw);
        }
        if (a.bc == BC_CAVITY && y == ny - 1) {
            if (xin) push_lid<ST, (NT & 2) != 0>(dst, P, x, y, pitch, in, ref, a.fp16_scale);
            continue;
        }
        const int fl = node9_row<ST, CO>(f, xs, y, nx, ny, a.bc, in);
        if (xin && (fl & 1)) bad = min(bad, y * nx + x);
        guarded += __popcll(__ballot(xin && (fl & 2)));
        if (xin) push9_xy<ST, (NT & 2) != 0>(dst, P, x, y, pitch, f, ref, a.fp16_scale);
    }
    report(a.status, bad, guarded, a.step, a.step_base);
}

// --------------------------------------------------------------------------
// D2Q9, one lattice, two steps per launch (temporal blocking).
//
// A block of BX threads owns an output tile of BX columns and H rows (in a
// batch, of the instance's tile width tw <= BX, below).  It walks a window
// that is one node wider on every side: window column i is
// lattice column x0 - 1 + i and window row j is lattice row y0 - 1 + j, each
// mapped into the lattice by the neighbour rule (wrapped on periodic axes,
// clamped otherwise).  The first step computes every window node exactly as
// the single-step kernels compute that lattice node, and rounds it to the
// storage type into LDS; the second step computes the tile's own nodes from
// those values and writes them to HBM.  Because the window rows and columns
// around a node are precisely its neighbour rows and columns, every result
// is bitwise equal to two single-step launches, while HBM sees one read and
// one write of each population per two steps.
//
// The first step runs row by row (thread t: column x0 + t) and the second
// step trails it by one row.  RS = 4 or 3 keeps all nine planes of a window
// row in a ring of RS rows: with four slots one barrier per row suffices (the
// row written in iteration j + 1 was last read in iteration j - 1); three
// take less LDS and a second barrier.  RS = 0 splits the planes by how long
// they are needed: the second step reads the unshifted planes 0, 2 and 4 only
// in the thread's own column, so they stay in registers (plane 4 of the row
// just computed, plane 0 of the row before, plane 2 of the row before that);
// planes 7 and 8 are read in the iteration that writes them (two slots),
// 1 and 3 one iteration later (three), 5 and 6 two iterations later (four).
// That is 18 plane-rows of LDS instead of 36, with one barrier per row.  The
// two halo columns of every window row are computed first, by the first
// 2 (H + 2) threads, into their own LDS array, and copied into the ring as
// each row is written.  The second step reads a halo column only in the three
// planes that stream in from that side (1, 5, 8 from the left; 3, 6, 7 from
// the right), so the array keeps those six values per row.  Each first-step row's loads are
// issued one iteration ahead, before the barrier, and complete during the
// second step of the row before.
// Only nodes inside the tile report status (first step at a.step, second at
// a.step + 1), so every node reports once per step.
// --------------------------------------------------------------------------

// Plane-rows of LDS the ring of the two-step kernel holds (RS as there).
constexpr int t2_plane_rows(int rs) { return rs == 0 ? 18 : 9 * rs; }

// LDS of the two-step kernel: the ring (plane-rows of bx + 2 columns) and
// the three planes the second step reads in each halo column of every window
// row.
template <class T>
constexpr size_t t2_lds_bytes(int bx, int h, int rs)
{
    return sizeof(T) * (size_t)(t2_plane_rows(rs) * (bx + 2) + 6 * (h + 2));
}

// Plane of the k-th value (k < 3) kept for a halo column: the left column
// (side 0) feeds planes 1, 5 and 8 of the tile's first column, the right one
// planes 3, 6 and 7 of its last.
__device__ __forceinline__ int t2_halo_plane(int side, int k)
{
    return side ? (k == 0 ? 3 : (k == 1 ? 6 : 7)) : (k == 0 ? 1 : (k == 1 ? 5 : 8));
}

// Lattice coordinate of window coordinate g on an axis of n nodes: the
// neighbour rule one node beyond either edge (wrap or clamp); coordinates
// further out (ragged last tiles) are clamped, and those nodes are computed
// but never read.
__device__ __forceinline__ int t2_map(int g, int n, bool wrap)
{
    if (g < 0) return wrap ? n - 1 : 0;
    if (g >= n) return (wrap && g == n) ? 0 : n - 1;
    return g;
}

// LDS bytes of one wave's tile in the wave-tiled mode (64 columns), rounded
// to 16 bytes.
template <class T>
constexpr size_t t2_wave_lds_bytes(int h, int rs)
{
    return (t2_lds_bytes<T>(64, h, rs) + 15) / 16 * 16;
}

// WT > 0 (batches): wave-tiled mode.  Each of the block's WT waves owns a
// tile of 64 columns (BX = 64) from the tile table, with an LDS region of its
// own; the waves never wait for each other, and a wave without a tile leaves
// at once.
template <int ST, int CO, int BX, int H, int RS, int NT = 0, int WPE = 0, bool BATCH = false, int WT = 0>
__global__ __launch_bounds__(WT > 0 ? 64 * WT : BX) __attribute__((amdgpu_waves_per_eu(WPE > 0 ? WPE : 1)))
void k_d2q9_t2(const typename Form<ST>::T *__restrict__ src_all, typename Form<ST>::T *__restrict__ dst_all,
               StepArgs a)
{
    using C = typename Form<ST>::C;
    using T = typename Form<ST>::T;
    constexpr int W = BX + 2;     // window columns
    extern __shared__ __align__(16) unsigned char t2_lds[];
    static_assert(RS == 0 || RS == 3 || RS == 4, "ring of three or four window rows, or split rings");
    static_assert(WT == 0 || (BATCH && BX == 64), "wave-tiled mode: batches, 64-column tiles");
    // Barrier between a row's LDS writes and their reads: the block's, or in
    // the wave-tiled mode the wave's own.
    auto sync = [] {
        if constexpr (WT > 0) lds_wave_sync();
        else lds_barrier();
    };
    // Tile-table entry of this block (or of this wave in the wave-tiled mode).
    // (The wave index is read from the first lane so that the compiler knows
    // it, and everything derived from the tile, to be wave-uniform.)
    const int wave = WT > 0 ? __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)) : 0;
    const int tile = WT > 0 ? (int)blockIdx.x * WT + wave
                            : (BATCH && a.xcd_swizzle ? xcd_remap((int)blockIdx.x, (int)gridDim.x) : (int)blockIdx.x);
    if constexpr (WT > 0) {
        if (tile >= a.ntiles) return;  // wave-uniform; no block barrier in this mode
    }
    T *ring = (T *)(t2_lds + (size_t)wave * (WT > 0 ? t2_wave_lds_bytes<T>(H, RS) : 0));
    // RS > 0: [RS][9][W]; RS = 0: planes 7,8 [2][2][W], 1,3 [3][2][W], 5,6 [4][2][W]
    T *halo = ring + t2_plane_rows(RS) * W;  // [H + 2][2][3]
    // Plane q of window row j in the ring (q and the ring layout are
    // compile-time, j is uniform).
    auto plane = [&](int q, int j) -> T * {
        if constexpr (RS != 0) {
            return ring + ((j % RS) * 9 + q) * W;
        } else {
            if (q == 7 || q == 8) return ring + ((j & 1) * 2 + (q - 7)) * W;
            if (q == 1 || q == 3) return ring + (4 + (j % 3) * 2 + (q == 3)) * W;
            return ring + (10 + (j & 3) * 2 + (q - 5)) * W;  // q = 5, 6
        }
    };
    // Instance and tile of this block: a single lattice's grid of tiles, or a
    // batch's tile table (instance, tile index within the instance).
    const int ii = BATCH ? a.tile_inst[tile] : 0;
    const Inst &in = BATCH ? a.inst[ii] : a.one;
    const int nx = in.nx, ny = in.ny, pitch = in.pitch;
    const int64_t P = in.plane;
    const int tiles_x = BATCH ? (nx + BX - 1) / BX : a.tiles_x;
    int tx, ty;
    if constexpr (BATCH) {
        const int k = a.tile_first[tile];
        ty = k / tiles_x;
        tx = k - ty * tiles_x;
    } else {
        tile_of_block(a.xcd_swizzle, a.tiles_x, tx, ty);
    }
    const T *src = src_all + (BATCH ? in.offset : 0);
    T *dst = dst_all + (BATCH ? in.offset : 0);
    DevStatus *status = a.status + ii;
    const bool xw = a.bc == BC_PERIODIC;
    const bool yw = a.bc == BC_PERIODIC || a.bc == BC_TUBE;
    const bool cavity = a.bc == BC_CAVITY;
    const int t = WT > 0 ? (int)(threadIdx.x & 63) : (int)threadIdx.x;
    // Tile width: BX, or in a batch the instance's columns spread evenly over
    // its tiles_x tiles, rounded up to whole waves (an instance 300 wide
    // takes two tiles of 192 columns instead of two of 256).  The waves of a
    // block that hold no needed column, beyond the tile's width or beyond the
    // column just past the instance's edge, skip the arithmetic and keep
    // every barrier.
    constexpr bool BAL = BATCH && WT == 0;
    int tw = BX;
    if constexpr (BAL) tw = min(BX, ((nx + tiles_x - 1) / tiles_x + 63) & ~63);
    const int x0 = tx * tw, y0 = ty * H;
    const int hn = min(H, ny - y0);  // output rows of this tile (block-uniform)
    const int x = x0 + t;
    const bool xin = (!BAL || t < tw) && x < nx;
    const int xs = t2_map(x, nx, xw);  // lattice column of this thread's window column
    bool wave_on = true;
    if constexpr (BAL) {
        const int t0 = __builtin_amdgcn_readfirstlane(t & ~63);
        wave_on = t0 < tw && t0 <= nx - x0;
    }

    // Steps this launch takes here (block-uniform): two; one for an odd step
    // count's last step, or for a batch instance whose step limit falls
    // between the two (the first step's own nodes then go straight to HBM);
    // none for a stopped instance, which carries its state over.
    int kdo = a.max_steps;
    if constexpr (BATCH) {
        const int64_t s0 = a.step + (a.step_base ? *a.step_base : 0);
        kdo = (int)max((int64_t)0, min((int64_t)kdo, in.stop - s0));
    }
    if (kdo <= 0) {
        if (xin)
            for (int r = 0; r < hn; ++r) carry_node(src, dst, P, 9, (y0 + r) * pitch + x);
        return;
    }
    const Cols cols = columns(xs, tx == 0 || tx == tiles_x - 1, nx, a.bc, sizeof(T));
    C ref[9];
    ref9<C>(C(in.rho0), ref);

    // The first window row's loads are issued first, so that they are in
    // flight during the halo columns' first step.
    const int nj = hn + 2;
    auto row_of = [&](int j) { return t2_map(y0 - 1 + j, ny, yw); };
    auto pull_row = [&](int j, T (&r)[9]) {
        const int gy = row_of(j);
        if (cavity && gy == ny - 1) return;  // the lid row loads nothing
        const Nb n = neighbours(0, gy, 1, ny, a.bc);  // rows only
        pull9_row_u<ST, nl_mode(NT)>(src, P, gy, n.ym, n.yp, pitch, cols.cc, cols.cm, cols.cp, r);
    };
    T raw[9];
    if (wave_on) pull_row(0, raw);

    // Halo columns (x0 - 1 and x0 + tw) of every window row, first step.
    for (int k = t; k < 2 * (hn + 2); k += BX) {
        const int side = k & 1, j = k >> 1;
        const int gx = t2_map(side ? x0 + tw : x0 - 1, nx, xw);
        const int gy = row_of(j);
        C f[9];
        const Nb n = neighbours(gx, gy, nx, ny, a.bc);
        pull9<ST>(src, P, gx, gy, pitch, n, ref, a.fp16_iscale, f);
        (void)node9<ST, CO>(f, role9(gx, gy, nx, ny, a.bc), in);
        // The three planes the second step reads in this column (t2_halo_plane;
        // ref is the same within the axis and within the diagonal directions).
        T *h = halo + (j * 2 + side) * 3;
        store<ST>(h + 0, side ? f[3] : f[1], ref[1], a.fp16_scale);
        store<ST>(h + 1, side ? f[6] : f[5], ref[5], a.fp16_scale);
        store<ST>(h + 2, side ? f[7] : f[8], ref[5], a.fp16_scale);
    }

    int bad1 = kNoNode, bad2 = kNoNode;
    int guarded = 0;
    if constexpr (BAL) {
        if (!wave_on) {
            // A wave without a needed column takes only the block's barriers,
            // as many and in the order the row loop below takes them.
            sync();  // halo array complete
            for (int j = 0; j < nj; ++j) {
                if constexpr (RS == 3) {
                    if (j > 0) sync();
                }
                sync();
            }
            return;
        }
    }
    T lid_st[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) lid_st[q] = to_storage_apart<ST>(C(in.lid[q]), ref[q], a.fp16_scale);
    sync();  // halo array complete

    // Iteration j: first step of window row j from raw (loaded in the
    // iteration before), loads of row j + 1 into raw, barrier, second step of
    // lattice row y0 + j - 2.
    constexpr int kShifted[6] = {1, 3, 5, 6, 7, 8};  // planes read in a neighbour column
    T u0 = T(0), u2a = T(0), u2b = T(0);  // RS = 0: plane 0 of row j - 1, plane 2 of rows j - 1 and j - 2
    for (int j = 0; j < nj; ++j) {
        // Three slots: the slot written now was read by the last second step.
        if constexpr (RS == 3) {
            if (j > 0) sync();
        }
        T v0 = T(0), v2 = T(0), v4 = T(0);  // RS = 0: the unshifted planes of row j
        {
            const int gy = row_of(j);
            // The row's populations in storage form, converted once for the
            // ring and the direct write: the lid row's are the lid
            // equilibrium's (uniform), any other row's its first step's.
            T sv[9];
            int fl = 0;
            if (cavity && gy == ny - 1) {
                // (An empty statement gives this path a block of its own, so
                // that the copies below are not hoisted onto every row.)
                asm volatile("");
#pragma unroll
                for (int q = 0; q < 9; ++q) sv[q] = lid_st[q];
            } else {
                C f[9];
#pragma unroll
                for (int q = 0; q < 9; ++q) f[q] = load<ST>(&raw[q], ref[q], a.fp16_iscale);
                fl = node9_row<ST, CO>(f, xs, gy, nx, ny, a.bc, in);
#pragma unroll
                for (int q = 0; q < 9; ++q) sv[q] = to_storage<ST>(f[q], ref[q], a.fp16_scale);
            }
            const bool own = j >= 1 && j <= hn && xin;
            if (own && (fl & 1)) bad1 = min(bad1, gy * nx + x);
            guarded += __popcll(__ballot(own && (fl & 2)));
            if (kdo == 1 && own) push9_xy_st<ST, (NT & 2) != 0>(dst, P, x, gy, pitch, sv);
            if constexpr (RS != 0) {
#pragma unroll
                for (int q = 0; q < 9; ++q) plane(q, j)[t + 1] = sv[q];
                if (t < 6) {
                    const int side = t >= 3, k = t - 3 * side;
                    plane(t2_halo_plane(side, k), j)[side ? tw + 1 : 0] = halo[(j * 2 + side) * 3 + k];
                }
            } else {
#pragma unroll
                for (int k = 0; k < 6; ++k) {
                    const int q = kShifted[k];
                    plane(q, j)[t + 1] = sv[q];
                }
                v0 = sv[0];
                v2 = sv[2];
                v4 = sv[4];
                if (t < 6) {
                    const int side = t >= 3, k = t - 3 * side;
                    plane(t2_halo_plane(side, k), j)[side ? tw + 1 : 0] = halo[(j * 2 + side) * 3 + k];
                }
            }
        }
        if (j + 1 < nj) pull_row(j + 1, raw);  // completes during this second step
        sync();
        // Unshifted planes this second step reads from registers (rows j - 1
        // and j - 2), then the delay line moves on by one row.
        const T s0 = u0, s2 = u2b;
        u0 = v0;
        u2b = u2a;
        u2a = v2;
        if (j < 2 || kdo == 1) continue;
        // Second step, lattice row y = y0 + j - 2 (window row j - 1): window
        // rows j - 2 and j hold its neighbour rows, window columns t and
        // t + 2 its neighbour columns.
        const int y = y0 + j - 2;
        if (cavity && y == ny - 1) {
            if (xin) push_lid<ST, (NT & 2) != 0>(dst, P, x, y, pitch, in, ref, a.fp16_scale);
            continue;
        }
        C f[9];
        if constexpr (RS != 0) {
            f[0] = load<ST>(plane(0, j - 1) + t + 1, ref[0], a.fp16_iscale);
            f[2] = load<ST>(plane(2, j - 2) + t + 1, ref[2], a.fp16_iscale);
            f[4] = load<ST>(plane(4, j) + t + 1, ref[4], a.fp16_iscale);
        } else {
            f[0] = load<ST>(&s0, ref[0], a.fp16_iscale);
            f[2] = load<ST>(&s2, ref[2], a.fp16_iscale);
            f[4] = load<ST>(&v4, ref[4], a.fp16_iscale);
        }
        f[1] = load<ST>(plane(1, j - 1) + t, ref[1], a.fp16_iscale);
        f[3] = load<ST>(plane(3, j - 1) + t + 2, ref[3], a.fp16_iscale);
        f[5] = load<ST>(plane(5, j - 2) + t, ref[5], a.fp16_iscale);
        f[6] = load<ST>(plane(6, j - 2) + t + 2, ref[6], a.fp16_iscale);
        f[7] = load<ST>(plane(7, j) + t + 2, ref[7], a.fp16_iscale);
        f[8] = load<ST>(plane(8, j) + t, ref[8], a.fp16_iscale);
        const int fl = node9_row<ST, CO>(f, xs, y, nx, ny, a.bc, in);
        if (xin && (fl & 1)) bad2 = min(bad2, y * nx + x);
        guarded += __popcll(__ballot(xin && (fl & 2)));
        if (xin) push9_xy<ST, (NT & 2) != 0>(dst, P, x, y, pitch, f, ref, a.fp16_scale);
    }
    report(status, bad1, guarded, a.step, a.step_base);
    report(status, bad2, 0, a.step + 1, a.step_base);
}

// --------------------------------------------------------------------------
// D2Q9, batch of lattices.  A tile is BLK consecutive nodes (row-major) of
// one instance; tile tables give its instance and first node.
// --------------------------------------------------------------------------

template <int ST, int CO, int BLK, int NT = 0>
__global__ __launch_bounds__(BLK) void k_d2q9_batch(const typename Form<ST>::T *__restrict__ src,
                                                    typename Form<ST>::T *__restrict__ dst, StepArgs a)
{
    using C = typename Form<ST>::C;
    if constexpr ((NT & 8) != 0) __builtin_amdgcn_s_setprio(2);  // until the loads are issued
    int t = blockIdx.x;
    if (a.xcd_swizzle) t = xcd_remap(t, gridDim.x);
    const int i = a.tile_inst[t];
    const Inst &in = a.inst[i];
    const int nx = in.nx, ny = in.ny;
    const int64_t P = in.plane;
    const int nodes = nx * ny;
    int node = a.tile_first[t] + (int)threadIdx.x;
    const bool valid = node < nodes;
    if (!valid) node = nodes - 1;
    // node -> (x, y): float estimate, exact after one correction (node < 2^24).
    int y = (int)((float)node * __builtin_amdgcn_rcpf((float)nx));
    int x = node - y * nx;
    if (x < 0) { --y; x += nx; }
    if (x >= nx) { ++y; x -= nx; }
    constexpr uint32_t E = sizeof(typename Form<ST>::T);
    // Byte offsets of the node's row and its rows below and above (rows are
    // `pitch` elements apart; the neighbours are one row away unless the
    // wrap/clamp rule applies).
    const uint32_t rb = (uint32_t)in.pitch * E, rc = (uint32_t)y * rb;
    if (instance_stopped(a, in)) {  // uniform across the block
        if (valid) carry_node(src + in.offset, dst + in.offset, P, 9, y * in.pitch + x);
        return;
    }
    C ref[9];
    ref9<C>(C(in.rho0), ref);
    const Nb n = neighbours(x, y, nx, ny, a.bc);
    const uint32_t rm = n.ym == y - 1 ? rc - rb : (uint32_t)n.ym * rb;
    const uint32_t rp = n.yp == y + 1 ? rc + rb : (uint32_t)n.yp * rb;
    C f[9];
    {
        typename Form<ST>::T raw[9];
        pull9_inst<ST, nl_mode(NT)>(uniform_addr(src + in.offset), P, rc, rm, rp, (uint32_t)x * E,
                                    (uint32_t)n.xm * E, (uint32_t)n.xp * E, raw);
        if constexpr ((NT & 8) != 0) __builtin_amdgcn_s_setprio(0);
#pragma unroll
        for (int q = 0; q < 9; ++q) f[q] = load<ST>(&raw[q], ref[q], a.fp16_iscale);
    }
    const int role = role9(x, y, nx, ny, a.bc);
    const int fl = node9<ST, CO>(f, role, in);
    if (valid)
        push9_inst<ST, (NT & 2) != 0>(uniform_addr(dst + in.offset), P, rc + (uint32_t)x * E, f, ref,
                                      a.fp16_scale);
    const int guarded = __popcll(__ballot(valid && (fl & 2)));
    report(a.status + i, valid && (fl & 1) ? node : kNoNode, guarded, a.step, a.step_base);
}

// --------------------------------------------------------------------------
// D2Q9, batch of small lattices resident in LDS: one workgroup per instance
// runs `nsteps` steps inside one launch.  Both population buffers live in
// LDS at storage precision (so every step rounds exactly as the per-step
// kernels do and results are bitwise identical); one workgroup barrier
// separates the steps.  The state is read from `src` once and the final
// state written to `dst` once (they may be the same buffer: every read
// happens before the first write).
//
// A step takes as long as the collisions that one SIMD issues (1,550 cycles a
// wave, MinxEnt4 FP64), so the nodes that collide come first, packed into as few
// waves as hold them, and the wall nodes last, in waves that only swap: 17^2
// cavities are four collision waves, one on each SIMD, and one wave of walls,
// where row-major order has five that all collide.  A thread keeps its node's
// ten LDS addresses and its role over all steps if the block has a thread
// for every node.  Against row-major nodes, placed anew at each step (us per
// step): 300 cavities of 17^2 FP64 MinxEnt4 3.20 -> 2.07 (44 compute units hold
// two), FP32 1.84 -> 1.30, SRT FP64 1.57 -> 1.02; 256 of 32^2 FP64 3.80 -> 3.35;
// 300 of 33^2, more nodes than threads, 8.00 -> 6.86.
// --------------------------------------------------------------------------

// Node `idx` of a lattice in that order: the fluid rectangle row by row, the
// walls below it, on its left and right, and above it.
struct LdsNode {
    int x, y;
};

__device__ __forceinline__ LdsNode lds_node(int idx, int nx, int ny, int bc)
{
    const int wx = bc == BC_PERIODIC ? 0 : 1, wy = bc == BC_CAVITY || bc == BC_BOX ? 1 : 0;
    const int fx = nx - 2 * wx, fy = ny - 2 * wy, fluid = fx * fy;
    // Quotients of indices below 2^13 by a float estimate, exact after one
    // correction.
    auto split = [](int i, int w, int &q, int &r) {
        q = (int)((float)i * __builtin_amdgcn_rcpf((float)w));
        r = i - q * w;
        if (r < 0) { --q; r += w; }
        if (r >= w) { ++q; r -= w; }
    };
    LdsNode n;
    if (idx < fluid) {
        split(idx, fx, n.y, n.x);
        n.x += wx;
        n.y += wy;
        return n;
    }
    const int i = idx - fluid, below = wy * nx, sides = 2 * fy;
    if (i < below) {
        n.x = i;
        n.y = 0;
    } else if (i < below + sides) {
        n.x = (i - below) & 1 ? nx - 1 : 0;
        n.y = wy + ((i - below) >> 1);
    } else {
        n.x = i - below - sides;
        n.y = ny - 1;
    }
    return n;
}

template <int ST, int CO>
__global__ __launch_bounds__(1024) void k_d2q9_lds(const typename Form<ST>::T *src, typename Form<ST>::T *dst,
                                                   StepArgs a, int nsteps)
{
    using C = typename Form<ST>::C;
    using T = typename Form<ST>::T;
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int i = blockIdx.x;
    const Inst &tab = a.inst[i];
    const int nx = tab.nx, ny = tab.ny;
    const int nodes = nx * ny;
    T *L = (T *)lds_raw;  // buffer b at element 9 * nodes * b
    const T *g = src + tab.offset;
    // LDS holds the nodes without the row padding: node j of plane q at
    // q * nodes + j.
    for (int idx = threadIdx.x; idx < 9 * nodes; idx += blockDim.x) {
        const int q = idx / nodes, j = idx - q * nodes, jy = j / nx;
        L[idx] = g[q * tab.plane + jy * tab.pitch + (j - jy * nx)];
    }
    Inst in;  // what the collision reads
    in.omega = tab.omega;
    in.omega2 = tab.omega2;
    C ref[9];
    ref9<C>(C(tab.rho0), ref);
    const int64_t s0 = a.step + (a.step_base ? *a.step_base : 0);
    uint64_t first_bad = ~0ull;  // first step, smallest node of this thread
    int64_t guarded = 0;
    // Steps this instance takes in this launch (its step limit may end them
    // early; uniform across the block).
    const int kdone = (int)max((int64_t)0, min((int64_t)nsteps, tab.stop - s0));
    struct Place {
        int wr, rd[9], role;
    };
    auto place = [&](int idx) {
        const LdsNode n = lds_node(idx, nx, ny, a.bc);
        const Nb b = neighbours(n.x, n.y, nx, ny, a.bc);
        const int r = n.y * nx, rm = b.ym * nx, rp = b.yp * nx;
        const int o[9] = {r + n.x,  r + b.xm,  rm + n.x, r + b.xp, rp + n.x,
                          rm + b.xm, rm + b.xp, rp + b.xp, rp + b.xm};
        Place p;
        p.wr = o[0];
#pragma unroll
        for (int q = 0; q < 9; ++q) p.rd[q] = q * nodes + o[q];
        p.role = role9(n.x, n.y, nx, ny, a.bc);
        return p;
    };
    auto step = [&](const Place &p, int k) {
        const T *s = L + ((k & 1) ? 9 * nodes : 0);
        T *d = L + ((k & 1) ? 0 : 9 * nodes) + p.wr;
        C f[9];
        if (p.role == R_LID) {
#pragma unroll
            for (int q = 0; q < 9; ++q) f[q] = C(tab.lid[q]);
        } else {
#pragma unroll
            for (int q = 0; q < 9; ++q) f[q] = load<ST>(s + p.rd[q], ref[q], a.fp16_iscale);
            const int fl = node9<ST, CO>(f, p.role, in);
            if (fl & 1) first_bad = min(first_bad, event_key(s0 + k, p.wr));
            guarded += (fl >> 1) & 1;
        }
#pragma unroll
        for (int q = 0; q < 9; ++q) d[q * nodes] = to_storage<ST>(f[q], ref[q], a.fp16_scale);
    };
    __syncthreads();
    if (nodes <= (int)blockDim.x) {
        const bool has = (int)threadIdx.x < nodes;
        const Place p = place(has ? (int)threadIdx.x : 0);
        for (int k = 0; k < kdone; ++k) {
            if (has) step(p, k);
            lds_barrier();
        }
    } else {
        for (int k = 0; k < kdone; ++k) {
            for (int idx = threadIdx.x; idx < nodes; idx += blockDim.x) step(place(idx), k);
            lds_barrier();
        }
    }
    const T *fin = L + ((kdone & 1) ? 9 * nodes : 0);
    T *o = dst + tab.offset;
    for (int idx = threadIdx.x; idx < 9 * nodes; idx += blockDim.x) {
        const int q = idx / nodes, j = idx - q * nodes, jy = j / nx;
        o[q * tab.plane + jy * tab.pitch + (j - jy * nx)] = fin[idx];
    }
    // Status: rare events, one atomic per reporting lane.
    DevStatus *st = a.status + i;
    if (first_bad != ~0ull) {
        atomicOr(&st->flags, 1u);
        atomicMin((unsigned long long *)&st->first, (unsigned long long)first_bad);
    }
    if (guarded != 0) {
        atomicOr(&st->flags, 2u);
        atomicAdd((unsigned long long *)&st->guarded, (unsigned long long)guarded);
    }
}

template <int ST, int NT = 0>
__device__ __forceinline__ int step3_node(const typename Form<ST>::T *__restrict__ s,
                                          typename Form<ST>::T *__restrict__ d, int64_t P, int x, int nx,
                                          int bc, typename Form<ST>::C omega, typename Form<ST>::C rho0,
                                          const StepArgs &a, bool valid)
{
    using C = typename Form<ST>::C;
    const bool wrap = bc == BC_PERIODIC;
    const int xm = x > 0 ? x - 1 : (wrap ? nx - 1 : 0);
    const int xp = x < nx - 1 ? x + 1 : (wrap ? 0 : nx - 1);
    const C r0 = C(2.0 / 3.0) * rho0, r1 = C(1.0 / 6.0) * rho0;
    using T = typename Form<ST>::T;
    const T l0 = ldraw<T, (NT & 1) != 0>(s + x), l1 = ldraw<T, (NT & 1) != 0>(s + P + xm),
            l2 = ldraw<T, (NT & 1) != 0>(s + 2 * P + xp);
    C f0 = load<ST>(&l0, r0, a.fp16_iscale);
    C fp = load<ST>(&l1, r1, a.fp16_iscale);
    C fm = load<ST>(&l2, r1, a.fp16_iscale);
    const int role = (bc != BC_PERIODIC && (x == 0 || x == nx - 1)) ? R_WALL : R_FLUID;
    const int fl = node3<C>(f0, fp, fm, role, omega);
    if (valid) {
        store<ST, (NT & 2) != 0>(d + x, f0, r0, a.fp16_scale);
        store<ST, (NT & 2) != 0>(d + P + x, fp, r1, a.fp16_scale);
        store<ST, (NT & 2) != 0>(d + 2 * P + x, fm, r1, a.fp16_scale);
    }
    return fl;
}

// Eight consecutive populations moved as one or more 16-byte vector accesses.
template <class T, bool NT>
__device__ __forceinline__ void ld8(const T *p, T (&v)[8])
{
    constexpr int per = 16 / sizeof(T);
#pragma unroll
    for (int c = 0; c < 8 / per; ++c) {
        const u32x4 *q = (const u32x4 *)(p + c * per);
        u32x4 w;
        if constexpr (NT) w = __builtin_nontemporal_load(q);
        else w = *q;
        const Chunk<T> b = __builtin_bit_cast(Chunk<T>, w);
#pragma unroll
        for (int e = 0; e < per; ++e) v[c * per + e] = b.e[e];
    }
}

template <class T, bool NT>
__device__ __forceinline__ void st8(T *p, const T (&v)[8])
{
    constexpr int per = 16 / sizeof(T);
#pragma unroll
    for (int c = 0; c < 8 / per; ++c) {
        Chunk<T> b;
#pragma unroll
        for (int e = 0; e < per; ++e) b.e[e] = v[c * per + e];
        const u32x4 w = __builtin_bit_cast(u32x4, b);
        u32x4 *q = (u32x4 *)(p + c * per);
        if constexpr (NT) __builtin_nontemporal_store(w, q);
        else *q = w;
    }
}

// Eight consecutive nodes x0 .. x0+7 of one D1Q3 lattice (x0 a multiple of 8,
// x0 < nx; plane bases 256-byte aligned and plane lengths rounded up to 64
// elements, so each group is 16-byte aligned and inside its plane).  Every plane moves as
// 16-byte vectors; the two values shifted in from outside the group (plane 1
// from the left, plane 2 from the right) take one scalar load each, with the
// same wrap/clamp rule as the one-node form, so results are bitwise equal to
// it.  Nodes beyond nx in the last group are computed but neither stored nor
// counted.  Returns the smallest unstable valid node of the group, or kNoNode.
template <int ST, int NT = 0>
__device__ __forceinline__ int step3_group8(const typename Form<ST>::T *__restrict__ s,
                                             typename Form<ST>::T *__restrict__ d, int64_t P, int x0, int nx,
                                             int bc, typename Form<ST>::C omega, typename Form<ST>::C rho0,
                                             const StepArgs &a)
{
    using C = typename Form<ST>::C;
    using T = typename Form<ST>::T;
    constexpr bool NL = (NT & 1) != 0, NS = (NT & 2) != 0;
    T v0[8], v1[8], v2[8];
    ld8<T, NL>(s + x0, v0);
    ld8<T, NL>(s + P + x0, v1);
    ld8<T, NL>(s + 2 * P + x0, v2);
    const bool wrap = bc == BC_PERIODIC;
    const int jl = nx - 1 - x0 < 7 ? nx - 1 - x0 : 7;  // last valid node of the group
    const int xl = x0 + jl;
    const int xm = x0 > 0 ? x0 - 1 : (wrap ? nx - 1 : 0);
    const int xp = xl < nx - 1 ? xl + 1 : (wrap ? 0 : nx - 1);
    const T s1 = ldraw<T, NL>(s + P + xm), s2 = ldraw<T, NL>(s + 2 * P + xp);
    const C r0 = C(2.0 / 3.0) * rho0, r1 = C(1.0 / 6.0) * rho0;
    int bad = kNoNode;
    // Results go back into v0 and v2 in place (node j reads only v0[j] and
    // v2[j+1], not yet overwritten when walking upwards) but into o1 for
    // plane 1, whose node j reads v1[j-1].
    T o1[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int x = x0 + j;
        const T rp = j == 0 ? s1 : v1[j > 0 ? j - 1 : 0];
        const T rm = j < jl ? v2[j < 7 ? j + 1 : 7] : s2;
        C f0 = load<ST>(&v0[j], r0, a.fp16_iscale);
        C fp = load<ST>(&rp, r1, a.fp16_iscale);
        C fm = load<ST>(&rm, r1, a.fp16_iscale);
        const int role = (bc != BC_PERIODIC && (x == 0 || x == nx - 1)) ? R_WALL : R_FLUID;
        const int fl = node3<C>(f0, fp, fm, role, omega);
        if (bad == kNoNode && j <= jl && fl) bad = x;
        if constexpr (ST == ST_F16DEV) {
            v0[j] = enc16(f0, r0, a.fp16_scale);
            o1[j] = enc16(fp, r1, a.fp16_scale);
            v2[j] = enc16(fm, r1, a.fp16_scale);
        } else {
            v0[j] = T(f0);
            o1[j] = T(fp);
            v2[j] = T(fm);
        }
    }
    if (jl == 7) {
        st8<T, NS>(d + x0, v0);
        st8<T, NS>(d + P + x0, o1);
        st8<T, NS>(d + 2 * P + x0, v2);
    } else {
        for (int j = 0; j <= jl; ++j) {
            d[x0 + j] = v0[j];
            d[P + x0 + j] = o1[j];
            d[2 * P + x0 + j] = v2[j];
        }
    }
    return bad;
}

template <int ST, int BX, int NT = 0>
__global__ __launch_bounds__(BX) void k_d1q3_v8(const typename Form<ST>::T *__restrict__ src,
                                                typename Form<ST>::T *__restrict__ dst, StepArgs a)
{
    using C = typename Form<ST>::C;
    const Inst &in = a.one;
    const int x0 = (blockIdx.x * BX + (int)threadIdx.x) * 8;
    int bad = kNoNode;
    if (x0 < in.nx) bad = step3_group8<ST, NT>(src, dst, in.plane, x0, in.nx, a.bc, C(in.omega), C(in.rho0), a);
    report(a.status, bad, 0, a.step, a.step_base);
}

template <int ST, int BLK, int NT = 0>
__global__ __launch_bounds__(BLK) void k_d1q3_batch_v8(const typename Form<ST>::T *__restrict__ src,
                                                       typename Form<ST>::T *__restrict__ dst, StepArgs a)
{
    using C = typename Form<ST>::C;
    int t = blockIdx.x;
    if (a.xcd_swizzle) t = xcd_remap(t, gridDim.x);
    const int i = a.tile_inst[t];
    const Inst &in = a.inst[i];
    const int x0 = a.tile_first[t] + (int)threadIdx.x * 8;
    if (instance_stopped(a, in)) {  // uniform across the block
        for (int j = 0; j < 8 && x0 + j < in.nx; ++j)
            carry_node(src + in.offset, dst + in.offset, in.plane, 3, x0 + j);
        return;
    }
    int bad = kNoNode;
    if (x0 < in.nx)
        bad = step3_group8<ST, NT>(src + in.offset, dst + in.offset, in.plane, x0, in.nx, a.bc, C(in.omega),
                                   C(in.rho0), a);
    report(a.status + i, bad, 0, a.step, a.step_base);
}

template <int ST, int BX, int NPT, int NT = 0>
__global__ __launch_bounds__(BX) void k_d1q3(const typename Form<ST>::T *__restrict__ src,
                                             typename Form<ST>::T *__restrict__ dst, StepArgs a)
{
    using C = typename Form<ST>::C;
    const Inst &in = a.one;
    const int nx = in.nx;
    int bad = kNoNode;
#pragma unroll
    for (int k = 0; k < NPT; ++k) {
        const int x = (blockIdx.x * NPT + k) * BX + (int)threadIdx.x;
        const bool valid = x < nx;
        const int fl = step3_node<ST, NT>(src, dst, in.plane, valid ? x : nx - 1, nx, a.bc, C(in.omega),
                                      C(in.rho0), a, valid);
        if (valid && fl) bad = min(bad, x);
    }
    report(a.status, bad, 0, a.step, a.step_base);
}

template <int ST, int BLK, int NPT, int NT = 0>
__global__ __launch_bounds__(BLK) void k_d1q3_batch(const typename Form<ST>::T *__restrict__ src,
                                                    typename Form<ST>::T *__restrict__ dst, StepArgs a)
{
    using C = typename Form<ST>::C;
    int t = blockIdx.x;
    if (a.xcd_swizzle) t = xcd_remap(t, gridDim.x);
    const int i = a.tile_inst[t];
    const Inst &in = a.inst[i];
    const int nx = in.nx;
    if (instance_stopped(a, in)) {  // uniform across the block
        for (int k = 0; k < NPT; ++k) {
            const int x = a.tile_first[t] + k * BLK + (int)threadIdx.x;
            if (x < nx) carry_node(src + in.offset, dst + in.offset, in.plane, 3, x);
        }
        return;
    }
    int bad = kNoNode;
#pragma unroll
    for (int k = 0; k < NPT; ++k) {
        const int x = a.tile_first[t] + k * BLK + (int)threadIdx.x;
        const bool valid = x < nx;
        const int fl = step3_node<ST, NT>(src + in.offset, dst + in.offset, in.plane, valid ? x : nx - 1, nx, a.bc,
                                      C(in.omega), C(in.rho0), a, valid);
        if (valid && fl) bad = min(bad, x);
    }
    report(a.status + i, bad, 0, a.step, a.step_base);
}

// --------------------------------------------------------------------------
// State set-up and read-back (off the hot loop; FP64 in and out).
// --------------------------------------------------------------------------

// Node of a range of consecutive global node numbers (the instances' nodes one
// after another): its instance and its number there.  The range of instances
// a block meets is found once for the block (scalar), so most lanes have
// nothing left to search.
__device__ __forceinline__ int find_instance(const int64_t *__restrict__ prefix, int lo, int hi, int64_t g)
{
    while (lo < hi) {  // the last i in [lo, hi] with prefix[i] <= g
        const int mid = (lo + hi + 1) >> 1;
        if (prefix[mid] <= g) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

struct RangeNode {
    int inst;
    int node;
};

__device__ __forceinline__ RangeNode range_node(const NodeRange &r, int64_t g)
{
    if (!r.inst) return {0, (int)g};
    const int64_t b0 = r.g0 + (int64_t)blockIdx.x * 256;
    const int64_t b1 = b0 + 255 < r.g1 ? b0 + 255 : r.g1 - 1;
    const int lo = find_instance(r.prefix, 0, r.n - 1, b0);
    const int i = find_instance(r.prefix, lo, find_instance(r.prefix, lo, r.n - 1, b1), g);
    return {i, (int)(g - r.prefix[i])};
}

// Velocity of direction a.
template <int B>
__device__ __forceinline__ int init_vx(int a)
{
    return B == 9 ? cx9(a) : (a == 1 ? 1 : (a == 2 ? -1 : 0));
}
template <int B>
__device__ __forceinline__ int init_vy(int a)
{
    return B == 9 ? cy9(a) : 0;
}

// State set-up from the fields (or populations: b planes per instance) of
// nodes [g0, g1).  Storage slot (a, s) keeps what node s + v_a pulls next: node
// j therefore writes its own value of direction a to the slot of j - v_a, and
// to its own slot where j + v_a lies outside the lattice.  Every slot is
// written once and every field read once.  One lattice (not BATCH) is read from
// the kernel arguments, which keeps its sizes and addresses in scalar registers,
// and all loads come before the first store (us of whole calls, with one way
// for both and a load before each store / so: 32^2 fields set and read without
// allocation 35.9 / 32.4, lbm_set_populations 17^2 32.3 / 26.8, 128^2 90 / 81).
template <int ST, int B, bool BATCH>
__global__ __launch_bounds__(256) void k_init(NodeRange range, const double *__restrict__ rho,
                                              const double *__restrict__ ux, const double *__restrict__ uy,
                                              const double *__restrict__ fin, typename Form<ST>::T *buf,
                                              float scale)
{
    using C = typename Form<ST>::C;
    const int64_t g = range.g0 + (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (g >= range.g1) return;
    RangeNode rn = {0, (int)g};
    if constexpr (BATCH) rn = range_node(range, g);
    const Inst &in = BATCH ? range.inst[rn.inst] : range.one;
    const int64_t i = g - range.g0;  // of the field arrays
    const int nx = in.nx, ny = in.ny, bc = range.bc;
    const int j = rn.node;
    const double *fi = fin ? fin + B * (g - j) : nullptr;
    const int x = j % nx, y = j / nx;
    const bool xw = bc == BC_PERIODIC;
    const bool yw = (bc == BC_PERIODIC || bc == BC_TUBE) && B == 9;
    typename Form<ST>::T *d = buf + in.offset;
    const bool lid = B == 9 && bc == BC_CAVITY && y == ny - 1;
    double v[B];
    if (fin) {
#pragma unroll
        for (int a = 0; a < B; ++a) v[a] = fi[(int64_t)a * nx * ny + j];
    } else if (lid) {
#pragma unroll
        for (int a = 0; a < B; ++a) v[a] = in.lid[a];
    } else {
        const double r = rho[i], u = ux[i], w = B == 9 ? uy[i] : 0.0;
#pragma unroll
        for (int a = 0; a < B; ++a) {
            const double cu = init_vx<B>(a) * u + init_vy<B>(a) * w;
            const double wa = (B == 9) ? ((a == 0) ? 4.0 / 9.0 : (a < 5 ? 1.0 / 9.0 : 1.0 / 36.0))
                                       : (a == 0 ? 2.0 / 3.0 : 1.0 / 6.0);
            v[a] = wa * r * (1.0 + 3.0 * cu + 4.5 * cu * cu - 1.5 * (u * u + w * w));
        }
    }
#pragma unroll
    for (int a = 0; a < B; ++a) {
        const int vx = init_vx<B>(a), vy = init_vy<B>(a);
        C ref;
        if (B == 9) {
            ref = (a == 0 ? W9<C>::rest : (a < 5 ? W9<C>::axis : W9<C>::diag)) * C(in.rho0);
        } else {
            ref = (a == 0 ? C(2.0 / 3.0) : C(1.0 / 6.0)) * C(in.rho0);
        }
        typename Form<ST>::T *p = d + (int64_t)a * in.plane;
        int sx = x - vx, sy = y - vy;  // the node this one pulls direction a from
        if (xw) sx = sx < 0 ? sx + nx : (sx >= nx ? sx - nx : sx);
        if (yw) sy = sy < 0 ? sy + ny : (sy >= ny ? sy - ny : sy);
        if (sx >= 0 && sx < nx && sy >= 0 && sy < ny) store<ST>(p + (int64_t)sy * in.pitch + sx, C(v[a]), ref, scale);
        const int tx = x + vx, ty = y + vy;
        const bool out = (!xw && (tx < 0 || tx >= nx)) || (!yw && (ty < 0 || ty >= ny));
        if (out) store<ST>(p + (int64_t)y * in.pitch + x, C(v[a]), ref, scale);
    }
}

// Moments or populations of nodes [g0, g1), written from the first element of
// the output arrays on (device memory, or host memory the device can write:
// 55 GB/s over the link, the rate of its copy engines).
template <int ST, int B>
__global__ __launch_bounds__(256) void k_gather(NodeRange range, const typename Form<ST>::T *__restrict__ buf,
                                                double *rho, double *ux, double *uy, double *fout, int64_t fstride,
                                                float iscale)
{
    using C = typename Form<ST>::C;
    const int64_t g = range.g0 + (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (g >= range.g1) return;
    const RangeNode rn = range_node(range, g);
    const Inst &in = range.inst ? range.inst[rn.inst] : range.one;
    const int64_t i = g - range.g0;  // of the output arrays
    const int nx = in.nx, ny = in.ny, bc = range.bc;
    const int x = rn.node % nx, y = rn.node / nx;
    const int pitch = in.pitch;
    const typename Form<ST>::T *s = buf + in.offset;
    double f[9];
    if (B == 9) {
        C ref[9];
        ref9<C>(C(in.rho0), ref);
        C h[9];
        pull9<ST>(s, in.plane, x, y, pitch, neighbours(x, y, nx, ny, bc), ref, iscale, h);
        for (int a = 0; a < 9; ++a) f[a] = double(h[a]);
    } else {
        const bool wrap = bc == BC_PERIODIC;
        const int xm = x > 0 ? x - 1 : (wrap ? nx - 1 : 0);
        const int xp = x < nx - 1 ? x + 1 : (wrap ? 0 : nx - 1);
        const C r0 = C(2.0 / 3.0) * C(in.rho0), r1 = C(1.0 / 6.0) * C(in.rho0);
        f[0] = double(load<ST>(s + x, r0, iscale));
        f[1] = double(load<ST>(s + in.plane + xm, r1, iscale));
        f[2] = double(load<ST>(s + 2 * in.plane + xp, r1, iscale));
    }
    if (fout) {
        for (int a = 0; a < B; ++a) fout[a * fstride + i] = f[a];
        return;
    }
    double r, jx, jy;
    if (B == 9) {
        r = f[0] + f[1] + f[2] + f[3] + f[4] + f[5] + f[6] + f[7] + f[8];
        jx = f[1] - f[3] + f[5] - f[6] - f[7] + f[8];
        jy = f[2] - f[4] + f[5] + f[6] - f[7] - f[8];
    } else {
        r = f[0] + f[1] + f[2];
        jx = f[1] - f[2];
        jy = 0.0;
    }
    if (rho) rho[i] = r;
    if (ux) ux[i] = jx / r;
    if (uy) uy[i] = jy / r;
}

// Each thread moves kCopyVec 16-byte vectors, one block-width apart, so every
// load instruction of a wave covers 1 KiB of contiguous memory and a thread
// has kCopyVec loads in flight before its first store.
constexpr int kCopyVec = 4;

__global__ __launch_bounds__(256) void k_copy(u32x4 *__restrict__ d, const u32x4 *__restrict__ s, size_t n)
{
    const size_t b0 = (size_t)blockIdx.x * (256 * kCopyVec);
    const size_t i0 = b0 + threadIdx.x;
    u32x4 v[kCopyVec];
    if (b0 + 256 * kCopyVec <= n) {  // whole block: no per-vector test, loads all in flight
#pragma unroll
        for (int j = 0; j < kCopyVec; ++j) v[j] = __builtin_nontemporal_load(s + i0 + (size_t)j * 256);
#pragma unroll
        for (int j = 0; j < kCopyVec; ++j) __builtin_nontemporal_store(v[j], d + i0 + (size_t)j * 256);
        return;
    }
#pragma unroll
    for (int j = 0; j < kCopyVec; ++j) {
        const size_t i = i0 + (size_t)j * 256;
        if (i < n) v[j] = __builtin_nontemporal_load(s + i);
    }
#pragma unroll
    for (int j = 0; j < kCopyVec; ++j) {
        const size_t i = i0 + (size_t)j * 256;
        if (i < n) __builtin_nontemporal_store(v[j], d + i);
    }
}

__global__ void k_step_base(int64_t *b, int64_t v, int add)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) *b = add ? *b + v : v;
}

__global__ void k_clear_status(DevStatus *st, int n)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) {
        st[i].flags = 0;
        st[i].pad = 0;
        st[i].first = ~0ull;
        st[i].guarded = 0;
    }
}

// --------------------------------------------------------------------------
// Launchers
// --------------------------------------------------------------------------

namespace {

struct Shape {
    int bx, by, rpt, swz;
    const char *name;
    int steps = 1;  // steps per launch
};

// Launch shapes of the single-lattice D2Q9 kernel.  Every shape computes the
// same per-node arithmetic, so results are bitwise identical.
constexpr Shape kShapes[] = {
    {256, 1, 1, 0, "256x1 rows=1 linear"},
    {256, 1, 1, 1, "256x1 rows=1 xcd"},
    {64, 4, 1, 1, "64x4 rows=1 xcd"},
    {256, 1, 1, 0, "256x1 rows=1 linear nt-load nt-store"},
    {256, 1, 1, 0, "256x1 rows=1 linear nt-store"},
    {256, 1, 1, 1, "256x1 rows=1 xcd nt-load nt-store"},
    {256, -1, 4, 1, "256 rows=4 pipelined xcd nt-load nt-store"},
    {64, 4, 2, 1, "64x4 rows=2 xcd nt-load nt-store"},
    {256, -1, 2, 1, "256 rows=2 pipelined xcd nt-load"},
    {128, -1, 4, 1, "128 rows=4 pipelined xcd nt-store"},
    {256, 1, 2, 1, "256x1 rows=2 xcd nt-load nt-store"},
    {256, 1, 1, 0, "256x1 rows=1 linear nt-load nt-store waves>=6"},
    {256, 1, 1, 0, "256x1 rows=1 linear nt-load nt-store waves>=8"},
    {256, 1, 1, 0, "256x1 rows=1 linear nt-store waves>=6"},
    {256, 1, 1, 1, "256x1 rows=1 xcd nt-load nt-store waves>=6"},
    {256, 1, 1, 0, "256x1 rows=1 linear nt-load nt-store waves>=7"},
    {256, 1, 1, 0, "256x1 rows=1 linear nt-load"},
    {128, 1, 1, 0, "128x1 rows=1 linear nt-load nt-store"},
    {512, 1, 1, 0, "512x1 rows=1 linear nt-load nt-store"},
    {256, -2, 1, 0, "256 LDS-staged rows=1 linear nt-store"},
    {256, 1, 1, 0, "256x1 rows=1 linear nt-load(unshifted planes) nt-store"},
    {256, 1, 1, 0, "256x1 rows=1 linear nt-load(unshifted planes) nt-store waves>=6"},
    {256, 1, 1, 0, "256x1 rows=1 linear nt-load(unshifted planes) nt-store waves>=8"},
    {256, 1, 1, 0, "256x1 rows=1 linear nt-load(unshifted planes) nt-store prio"},
    {256, 1, 1, 0, "256x1 rows=1 linear nt-load(unshifted planes) nt-store waves>=6 prio"},
    {256, 1, 1, 0, "256x1 rows=1 linear nt-load(unshifted planes) nt-store waves>=8 prio"},
    {256, 32, 1, 0, "two steps per launch, 256x32 tiles, nt-load(unshifted planes) nt-store", 2},
    {256, 16, 1, 0, "two steps per launch, 256x16 tiles, nt-load(unshifted planes) nt-store", 2},
    {256, 64, 1, 0, "two steps per launch, 256x64 tiles, nt-load(unshifted planes) nt-store", 2},
    {128, 32, 1, 0, "two steps per launch, 128x32 tiles, nt-load(unshifted planes) nt-store", 2},
    {512, 32, 1, 0, "two steps per launch, 512x32 tiles, nt-load(unshifted planes) nt-store", 2},
    {256, 32, 1, 0, "two steps per launch, 256x32 tiles, nt-store", 2},
    {256, 16, 1, 0, "two steps per launch, 256x16 tiles, 3-row ring, nt-load(unshifted planes) nt-store", 2},
    {256, 16, 1, 0, "two steps per launch, 256x16 tiles, 3-row ring, nt-load(unshifted planes) nt-store waves>=5", 2},
    {128, 16, 1, 0, "two steps per launch, 128x16 tiles, 3-row ring, nt-load(unshifted planes) nt-store waves>=5", 2},
    {256, 24, 1, 0, "two steps per launch, 256x24 tiles, 3-row ring, nt-load(unshifted planes) nt-store waves>=5", 2},
    {512, 16, 1, 0, "two steps per launch, 512x16 tiles, nt-load(unshifted planes) nt-store", 2},
    {256, 16, 1, 0, "two steps per launch, 256x16 tiles, split rings, nt-load(unshifted planes) nt-store", 2},
    {256, 32, 1, 0, "two steps per launch, 256x32 tiles, split rings, nt-load(unshifted planes) nt-store", 2},
    {256, 16, 1, 0, "two steps per launch, 256x16 tiles, split rings, nt-load(unshifted planes) nt-store waves>=4", 2},
    {256, 32, 1, 0, "two steps per launch, 256x32 tiles, split rings, nt-load(unshifted planes) nt-store waves>=4", 2},
    {512, 32, 1, 0, "two steps per launch, 512x32 tiles, split rings, nt-load(unshifted planes) nt-store waves>=4", 2},
    {1024, 32, 1, 0, "two steps per launch, 1024x32 tiles, split rings, nt-load(unshifted planes) nt-store waves>=4", 2},
    {0, 0, 1, 0, "on-chip windows, up to 4 steps per launch", 4},
    {0, 0, 1, 0, "on-chip windows, up to 6 steps per launch", 6},
    {0, 0, 1, 0, "on-chip windows, up to 8 steps per launch", 8},
    {0, 0, 1, 0, "on-chip windows, up to 16 steps per launch", 16},
    {0, 0, 1, 0, "on-chip windows, up to 64 steps per launch", 64},
    {0, 0, 1, 0, "register pipeline, 2 steps per launch", 2},
    {0, 0, 1, 0, "register pipeline, 3 steps per launch", 3},
    {0, 0, 1, 0, "register pipeline, 4 steps per launch", 4},
    {0, 8, 1, 0, "register pipeline, 2 steps per launch, 64x8 tiles", 2},
    {0, 8, 1, 0, "register pipeline, 3 steps per launch, 64x8 tiles", 3},
    {0, 8, 1, 0, "register pipeline, 4 steps per launch, 64x8 tiles", 4},
    {0, 16, 1, 0, "register pipeline, 2 steps per launch, 64x16 tiles", 2},
    {0, 16, 1, 0, "register pipeline, 3 steps per launch, 64x16 tiles", 3},
    {0, 16, 1, 0, "register pipeline, 4 steps per launch, 64x16 tiles", 4},
    {0, 32, 1, 0, "register pipeline, 2 steps per launch, 64x32 tiles", 2},
    {0, 32, 1, 0, "register pipeline, 3 steps per launch, 64x32 tiles", 3},
    {0, 32, 1, 0, "register pipeline, 4 steps per launch, 64x32 tiles", 4},
};

constexpr int kNumShapes = sizeof(kShapes) / sizeof(kShapes[0]);
constexpr int kMaxGridY = 65535;  // grid y limit; larger tile counts use a 1D grid
constexpr int kNumPipes = 12;     // the last shapes: register pipeline, every collision rule
constexpr int kFirstPipe = kNumShapes - kNumPipes;
constexpr int kNumWindows = 5;    // before them: on-chip windows, every collision rule
constexpr int kFirstWindow = kFirstPipe - kNumWindows;
constexpr int kNumOneOther = 3;   // the other collision rules instantiate the first three single-step shapes

// Entry of kShapes of shape v of a collision rule, or -1.
int shape_of(int coll, int v)
{
    if (v < 0) return -1;
    if (coll == CO_MINXENT4) return v < kNumShapes ? v : -1;
    if (v < kNumOneOther) return v;
    v += kFirstWindow - kNumOneOther;
    return v < kNumShapes ? v : -1;
}

template <int ST, int CO, int BX, int BY, int RPT, int NT = 0, int WPE = 0>
hipError_t go9(const void *src, void *dst, StepArgs a, int swz, hipStream_t s)
{
    using T = typename Form<ST>::T;
    const int tiles_x = (a.one.nx + BX - 1) / BX;
    const int tiles_y = (a.one.ny + BY * RPT - 1) / (BY * RPT);
    a.tiles_x = tiles_x;
    a.xcd_swizzle = swz;
    const dim3 grid = tiles_y <= kMaxGridY ? dim3(tiles_x, tiles_y) : dim3(tiles_x * tiles_y);
    hipLaunchKernelGGL((k_d2q9<ST, CO, BX, BY, RPT, NT, WPE>), grid, dim3(BX, BY), 0, s,
                       (const T *)src, (T *)dst, a);
    return hipGetLastError();
}

template <int ST, int CO, int BX, int RY, int NT = 0>
hipError_t go9st(const void *src, void *dst, StepArgs a, int swz, hipStream_t s)
{
    using T = typename Form<ST>::T;
    const int tiles_x = (a.one.nx + BX - 1) / BX;
    const int tiles_y = (a.one.ny + RY - 1) / RY;
    a.tiles_x = tiles_x;
    a.xcd_swizzle = swz;
    const dim3 grid = tiles_y <= kMaxGridY ? dim3(tiles_x, tiles_y) : dim3(tiles_x * tiles_y);
    hipLaunchKernelGGL((k_d2q9_stage<ST, CO, BX, RY, NT>), grid, dim3(BX), 0, s, (const T *)src, (T *)dst, a);
    return hipGetLastError();
}

template <int ST, int CO, int BX, int RPT, int NT = 0, int WPE = 0>
hipError_t go9pf(const void *src, void *dst, StepArgs a, int swz, hipStream_t s)
{
    using T = typename Form<ST>::T;
    const int tiles_x = (a.one.nx + BX - 1) / BX;
    const int tiles_y = (a.one.ny + RPT - 1) / RPT;
    a.tiles_x = tiles_x;
    a.xcd_swizzle = swz;
    const dim3 grid = tiles_y <= kMaxGridY ? dim3(tiles_x, tiles_y) : dim3(tiles_x * tiles_y);
    hipLaunchKernelGGL((k_d2q9_pf<ST, CO, BX, RPT, NT, WPE>), grid, dim3(BX), 0, s,
                       (const T *)src, (T *)dst, a);
    return hipGetLastError();
}

template <int ST, int CO, int BX, int H, int RS, int NT = 0, int WPE = 0>
hipError_t go9t2(const void *src, void *dst, StepArgs a, int swz, hipStream_t s)
{
    using T = typename Form<ST>::T;
    const int tiles_x = (a.one.nx + BX - 1) / BX;
    const int tiles_y = (a.one.ny + H - 1) / H;
    a.tiles_x = tiles_x;
    a.xcd_swizzle = swz;
    const dim3 grid = tiles_y <= kMaxGridY ? dim3(tiles_x, tiles_y) : dim3(tiles_x * tiles_y);
    hipLaunchKernelGGL((k_d2q9_t2<ST, CO, BX, H, RS, NT, WPE>), grid, dim3(BX), t2_lds_bytes<T>(BX, H, RS), s,
                       (const T *)src, (T *)dst, a);
    return hipGetLastError();
}

// LDS beyond the default 64 KiB must be allowed per kernel before launch
// (outside any stream capture): the FP64 two-step tiles need it.
template <int ST, int CO, int BX, int H, int RS, int NT = 0, int WPE = 0>
hipError_t prep9t2()
{
    using T = typename Form<ST>::T;
    constexpr size_t b = t2_lds_bytes<T>(BX, H, RS);
    if (b <= 65536) return hipSuccess;
    return hipFuncSetAttribute((const void *)k_d2q9_t2<ST, CO, BX, H, RS, NT, WPE>,
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)b);
}

// Two-step shapes of the single-lattice kernel (MinxEnt4): launch, or with
// `prep` only set the kernel's LDS limit.
template <int ST, int CO>
hipError_t dispatch9t2(int v, bool prep, const void *src, void *dst, const StepArgs &a, hipStream_t s)
{
#define LBM_T2(BX, H, RS, NT, WPE)                                                            \
    return prep ? prep9t2<ST, CO, BX, H, RS, NT, WPE>()                                       \
                : go9t2<ST, CO, BX, H, RS, NT, WPE>(src, dst, a, kShapes[v].swz, s)
    switch (v) {
    case 26: LBM_T2(256, 32, 4, 6, 0);
    case 27: LBM_T2(256, 16, 4, 6, 0);
    case 28: LBM_T2(256, 64, 4, 6, 0);
    case 29: LBM_T2(128, 32, 4, 6, 0);
    case 30: LBM_T2(512, 32, 4, 6, 0);
    case 31: LBM_T2(256, 32, 4, 2, 0);
    case 32: LBM_T2(256, 16, 3, 6, 0);
    case 33: LBM_T2(256, 16, 3, 6, 5);
    case 34: LBM_T2(128, 16, 3, 6, 5);
    case 35: LBM_T2(256, 24, 3, 6, 5);
    case 36: LBM_T2(512, 16, 4, 6, 0);
    case 37: LBM_T2(256, 16, 0, 6, 0);
    case 38: LBM_T2(256, 32, 0, 6, 0);
    case 39: LBM_T2(256, 16, 0, 6, 4);
    case 40: LBM_T2(256, 32, 0, 6, 4);
    case 41: LBM_T2(512, 32, 0, 6, 4);
    case 42: LBM_T2(1024, 32, 0, 6, 4);
    default: return hipErrorInvalidValue;
    }
#undef LBM_T2
}

template <int ST, int CO>
hipError_t dispatch9(int v, const void *src, void *dst, const StepArgs &a, hipStream_t s)
{
    const int swz = kShapes[v].swz;
    switch (v) {
    case 0: return go9<ST, CO, 256, 1, 1>(src, dst, a, swz, s);
    case 1: return go9<ST, CO, 256, 1, 1>(src, dst, a, swz, s);
    case 2: return go9<ST, CO, 64, 4, 1>(src, dst, a, swz, s);
    default: break;
    }
    if constexpr (CO == CO_MINXENT4) {
        switch (v) {
        case 3: return go9<ST, CO, 256, 1, 1, 3>(src, dst, a, swz, s);
        case 4: return go9<ST, CO, 256, 1, 1, 2>(src, dst, a, swz, s);
        case 5: return go9<ST, CO, 256, 1, 1, 3>(src, dst, a, swz, s);
        case 6: return go9pf<ST, CO, 256, 4, 3>(src, dst, a, swz, s);
        case 7: return go9<ST, CO, 64, 4, 2, 3>(src, dst, a, swz, s);
        case 8: return go9pf<ST, CO, 256, 2, 1>(src, dst, a, swz, s);
        case 9: return go9pf<ST, CO, 128, 4, 2>(src, dst, a, swz, s);
        case 10: return go9<ST, CO, 256, 1, 2, 3>(src, dst, a, swz, s);
        case 11: return go9<ST, CO, 256, 1, 1, 3, 6>(src, dst, a, swz, s);
        case 12: return go9<ST, CO, 256, 1, 1, 3, 8>(src, dst, a, swz, s);
        case 13: return go9<ST, CO, 256, 1, 1, 2, 6>(src, dst, a, swz, s);
        case 14: return go9<ST, CO, 256, 1, 1, 3, 6>(src, dst, a, swz, s);
        case 15: return go9<ST, CO, 256, 1, 1, 3, 7>(src, dst, a, swz, s);
        case 16: return go9<ST, CO, 256, 1, 1, 1>(src, dst, a, swz, s);
        case 17: return go9<ST, CO, 128, 1, 1, 3>(src, dst, a, swz, s);
        case 18: return go9<ST, CO, 512, 1, 1, 3>(src, dst, a, swz, s);
        case 19: return go9st<ST, CO, 256, 1, 2>(src, dst, a, swz, s);
        case 20: return go9<ST, CO, 256, 1, 1, 6>(src, dst, a, swz, s);
        case 21: return go9<ST, CO, 256, 1, 1, 6, 6>(src, dst, a, swz, s);
        case 22: return go9<ST, CO, 256, 1, 1, 6, 8>(src, dst, a, swz, s);
        case 23: return go9<ST, CO, 256, 1, 1, 14>(src, dst, a, swz, s);
        case 24: return go9<ST, CO, 256, 1, 1, 14, 6>(src, dst, a, swz, s);
        case 25: return go9<ST, CO, 256, 1, 1, 14, 8>(src, dst, a, swz, s);
        default: return dispatch9t2<ST, CO>(v, false, src, dst, a, s);
        }
    }
    return hipErrorInvalidValue;
}

template <int ST>
hipError_t dispatch9c(int coll, int v, const void *src, void *dst, const StepArgs &a, hipStream_t s)
{
    switch (coll) {
    case CO_MINXENT4: return dispatch9<ST, CO_MINXENT4>(v, src, dst, a, s);
    case CO_MINXENT2: return dispatch9<ST, CO_MINXENT2>(v, src, dst, a, s);
    case CO_SRT: return dispatch9<ST, CO_SRT>(v, src, dst, a, s);
    case CO_TRT: return dispatch9<ST, CO_TRT>(v, src, dst, a, s);
    case CO_MRT: return dispatch9<ST, CO_MRT>(v, src, dst, a, s);
    default: return hipErrorInvalidValue;
    }
}


// Two-step batch shapes: one block per tile of the tile table (a.ntiles).
template <int ST, int CO, int BX, int H, int RS, int NT = 0, int WPE = 0>
hipError_t go9bt2(const void *src, void *dst, const StepArgs &a, hipStream_t s)
{
    using T = typename Form<ST>::T;
    hipLaunchKernelGGL((k_d2q9_t2<ST, CO, BX, H, RS, NT, WPE, true>), dim3(a.ntiles), dim3(BX),
                       t2_lds_bytes<T>(BX, H, RS), s, (const T *)src, (T *)dst, a);
    return hipGetLastError();
}

template <int ST, int CO, int BX, int H, int RS, int NT = 0, int WPE = 0>
hipError_t prep9bt2()
{
    using T = typename Form<ST>::T;
    constexpr size_t b = t2_lds_bytes<T>(BX, H, RS);
    if (b <= 65536) return hipSuccess;
    return hipFuncSetAttribute((const void *)k_d2q9_t2<ST, CO, BX, H, RS, NT, WPE, true>,
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)b);
}

// Wave-tiled two-step batch shapes: WT waves per block, one 64-column tile
// each.
template <int ST, int CO, int H, int RS, int NT, int WT>
hipError_t go9bt2w(const void *src, void *dst, const StepArgs &a, hipStream_t s)
{
    using T = typename Form<ST>::T;
    const int blocks = (a.ntiles + WT - 1) / WT;
    hipLaunchKernelGGL((k_d2q9_t2<ST, CO, 64, H, RS, NT, 0, true, WT>), dim3(blocks), dim3(64 * WT),
                       WT * t2_wave_lds_bytes<T>(H, RS), s, (const T *)src, (T *)dst, a);
    return hipGetLastError();
}

template <int ST, int CO, int H, int RS, int NT, int WT>
hipError_t prep9bt2w()
{
    using T = typename Form<ST>::T;
    constexpr size_t b = WT * t2_wave_lds_bytes<T>(H, RS);
    if (b <= 65536) return hipSuccess;
    return hipFuncSetAttribute((const void *)k_d2q9_t2<ST, CO, 64, H, RS, NT, 0, true, WT>,
                               hipFuncAttributeMaxDynamicSharedMemorySize, (int)b);
}

// Two-step batch shapes 17-20 are 9, 14, 15 and 10 with the tile table read
// in XCD-banded order: block b takes the tile xcd_remap(b), so each XCD works
// through a contiguous band of the table and horizontally adjacent tiles (and,
// in narrow instances, vertically adjacent ones) share its L2, which serves
// the window lines they have in common.
constexpr int banded_base(int v) { return v == 17 ? 9 : v == 18 ? 14 : v == 19 ? 15 : v == 20 ? 10 : v; }

template <int ST, int CO>
hipError_t dispatch9bt2(int v, bool prep, const void *src, void *dst, const StepArgs &a, hipStream_t s)
{
    v = banded_base(v);
#define LBM_BT2W(H, RS, NT, WT) return prep ? prep9bt2w<ST, CO, H, RS, NT, WT>() : go9bt2w<ST, CO, H, RS, NT, WT>(src, dst, a, s)
    switch (v) {
    case 12: LBM_BT2W(16, 3, 6, 4);
    case 13: LBM_BT2W(16, 0, 6, 4);
    default: break;
    }
#undef LBM_BT2W
#define LBM_BT2(BX, H, RS, NT) return prep ? prep9bt2<ST, CO, BX, H, RS, NT>() : go9bt2<ST, CO, BX, H, RS, NT>(src, dst, a, s)
#define LBM_BT2B(BX, H, RS, NT, WPE) \
    return prep ? prep9bt2<ST, CO, BX, H, RS, NT, WPE>() : go9bt2<ST, CO, BX, H, RS, NT, WPE>(src, dst, a, s)
    switch (v) {
    case 9: LBM_BT2(64, 16, 3, 6);
    case 10: LBM_BT2(64, 16, 0, 6);
    case 11: LBM_BT2(256, 16, 4, 6);
    case 14: LBM_BT2(256, 16, 3, 6);
    case 15: LBM_BT2(256, 16, 0, 6);
    case 16: LBM_BT2B(256, 16, 3, 6, 5);
    case 21: LBM_BT2(128, 16, 3, 6);
    case 22: LBM_BT2(128, 16, 0, 6);
    default: return hipErrorInvalidValue;
    }
#undef LBM_BT2
#undef LBM_BT2B
}

template <int ST, int CO>
hipError_t dispatch9b(int v, const void *src, void *dst, const StepArgs &a_in, hipStream_t s)
{
    using T = typename Form<ST>::T;
    // Tiles run in launch order; shapes 5 and 6 are 3 and 4 with tiles in
    // XCD-banded order instead (measured slower, kept as candidates), and so
    // are the two-step shapes 17-20 (of 9, 14, 15 and 10).
    StepArgs a = a_in;
    a.xcd_swizzle = 0;
    if (v == 5 || v == 6) {
        a.xcd_swizzle = 1;
        v -= 2;
    }
    if (banded_base(v) != v) {
        a.xcd_swizzle = 1;
        v = banded_base(v);
    }
    switch (v) {
    case 0: hipLaunchKernelGGL((k_d2q9_batch<ST, CO, 256, 0>), dim3(a.ntiles), dim3(256), 0, s, (const T *)src, (T *)dst, a); break;
    case 1: hipLaunchKernelGGL((k_d2q9_batch<ST, CO, 128, 0>), dim3(a.ntiles), dim3(128), 0, s, (const T *)src, (T *)dst, a); break;
    case 2: hipLaunchKernelGGL((k_d2q9_batch<ST, CO, 256, 3>), dim3(a.ntiles), dim3(256), 0, s, (const T *)src, (T *)dst, a); break;
    case 3: hipLaunchKernelGGL((k_d2q9_batch<ST, CO, 256, 2>), dim3(a.ntiles), dim3(256), 0, s, (const T *)src, (T *)dst, a); break;
    case 4: hipLaunchKernelGGL((k_d2q9_batch<ST, CO, 256, 6>), dim3(a.ntiles), dim3(256), 0, s, (const T *)src, (T *)dst, a); break;
    case 7: hipLaunchKernelGGL((k_d2q9_batch<ST, CO, 256, 10>), dim3(a.ntiles), dim3(256), 0, s, (const T *)src, (T *)dst, a); break;
    case 8: hipLaunchKernelGGL((k_d2q9_batch<ST, CO, 256, 14>), dim3(a.ntiles), dim3(256), 0, s, (const T *)src, (T *)dst, a); break;
    default:
        if constexpr (CO == CO_MINXENT4) return dispatch9bt2<ST, CO>(v, false, src, dst, a, s);
        return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int ST>
hipError_t dispatch9bc(int coll, int v, const void *src, void *dst, const StepArgs &a, hipStream_t s)
{
    switch (coll) {
    case CO_MINXENT4: return dispatch9b<ST, CO_MINXENT4>(v, src, dst, a, s);
    case CO_MINXENT2: return dispatch9b<ST, CO_MINXENT2>(v, src, dst, a, s);
    case CO_SRT: return dispatch9b<ST, CO_SRT>(v, src, dst, a, s);
    case CO_TRT: return dispatch9b<ST, CO_TRT>(v, src, dst, a, s);
    case CO_MRT: return dispatch9b<ST, CO_MRT>(v, src, dst, a, s);
    default: return hipErrorInvalidValue;
    }
}

struct Shape3 {
    int bx, npt;
    const char *name;
    int steps = 1;  // steps per launch (at most)
};
constexpr Shape3 kShapes3[] = {
    {256, 1, "256 nodes=1"},
    {256, 4, "256 nodes=4"},
    {512, 2, "512 nodes=2"},
    {128, 4, "128 nodes=4"},
    {256, 4, "256 nodes=4 nt-load nt-store"},
    {256, 8, "256 groups of 8 nodes, 16-byte vectors"},
    {256, 8, "256 groups of 8 nodes, 16-byte vectors nt-load nt-store"},
    {128, 8, "128 groups of 8 nodes, 16-byte vectors nt-load nt-store"},
    // bx: nodes per lane
    {2, 0, "nodes in registers, 2 per lane, up to 32 steps per launch", 32},
    {4, 0, "nodes in registers, 4 per lane, up to 32 steps per launch", 32},
    {8, 0, "nodes in registers, 8 per lane, up to 32 steps per launch", 32},
};
constexpr int kFirstRegs3 = 8;
constexpr int kNumShapes3 = sizeof(kShapes3) / sizeof(kShapes3[0]);

template <int ST, int BX, int NT = 0>
hipError_t go3v(const void *src, void *dst, const StepArgs &a, hipStream_t s)
{
    using T = typename Form<ST>::T;
    const int groups = (a.one.nx + 7) / 8;
    hipLaunchKernelGGL((k_d1q3_v8<ST, BX, NT>), dim3((groups + BX - 1) / BX), dim3(BX), 0, s, (const T *)src,
                       (T *)dst, a);
    return hipGetLastError();
}

template <int ST, int BX, int NPT, int NT = 0>
hipError_t go3(const void *src, void *dst, const StepArgs &a, hipStream_t s)
{
    using T = typename Form<ST>::T;
    const int blocks = (a.one.nx + BX * NPT - 1) / (BX * NPT);
    hipLaunchKernelGGL((k_d1q3<ST, BX, NPT, NT>), dim3(blocks), dim3(BX), 0, s, (const T *)src, (T *)dst, a);
    return hipGetLastError();
}

template <int ST>
hipError_t dispatch3(int v, const void *src, void *dst, const StepArgs &a, hipStream_t s)
{
    switch (v) {
    case 0: return go3<ST, 256, 1>(src, dst, a, s);
    case 1: return go3<ST, 256, 4>(src, dst, a, s);
    case 2: return go3<ST, 512, 2>(src, dst, a, s);
    case 3: return go3<ST, 128, 4>(src, dst, a, s);
    case 4: return go3<ST, 256, 4, 3>(src, dst, a, s);
    case 5: return go3v<ST, 256>(src, dst, a, s);
    case 6: return go3v<ST, 256, 3>(src, dst, a, s);
    case 7: return go3v<ST, 128, 3>(src, dst, a, s);
    default:
        if (v >= kFirstRegs3 && v < kNumShapes3) return launch_d1q3_regs(ST, kShapes3[v].bx, 0, src, dst, a, s);
        return hipErrorInvalidValue;
    }
}

// Batched launch shapes: D2Q9 tiles of 256 or 128 nodes (one per thread);
// D1Q3 tiles of BLK x NPT nodes.
struct ShapeB {
    int blk, npt;
    const char *name;
    int steps = 1;  // steps per launch
    int rows = 0;   // two-step shapes: tile rows (tiles are blk x rows nodes of one instance)
};
constexpr ShapeB kShapesB9[] = {{256, 1, "batch 256 nodes/block"}, {128, 1, "batch 128 nodes/block"},
                                {256, 1, "batch 256 nodes/block nt-load nt-store"},
                                {256, 1, "batch 256 nodes/block nt-store"},
                                {256, 1, "batch 256 nodes/block nt-load(unshifted planes) nt-store"},
                                {256, 1, "batch 256 nodes/block nt-store, XCD-banded"},
                                {256, 1, "batch 256 nodes/block nt-load(unshifted planes) nt-store, XCD-banded"},
                                {256, 1, "batch 256 nodes/block nt-store prio"},
                                {256, 1, "batch 256 nodes/block nt-load(unshifted planes) nt-store prio"},
                                // two steps per launch (MinxEnt4 only)
                                {64, 1, "batch two steps per launch, 64x16 tiles, 3-row ring, nt-load(unshifted planes) nt-store", 2, 16},
                                {64, 1, "batch two steps per launch, 64x16 tiles, split rings, nt-load(unshifted planes) nt-store", 2, 16},
                                {256, 1, "batch two steps per launch, 256x16 tiles, nt-load(unshifted planes) nt-store", 2, 16},
                                {64, 1, "batch two steps per launch, 64x16 tiles one per wave (4 waves/block), 3-row ring, nt-load(unshifted planes) nt-store", 2, 16},
                                {64, 1, "batch two steps per launch, 64x16 tiles one per wave (4 waves/block), split rings, nt-load(unshifted planes) nt-store", 2, 16},
                                {256, 1, "batch two steps per launch, 256x16 tiles, 3-row ring, nt-load(unshifted planes) nt-store", 2, 16},
                                {256, 1, "batch two steps per launch, 256x16 tiles, split rings, nt-load(unshifted planes) nt-store", 2, 16},
                                {256, 1, "batch two steps per launch, 256x16 tiles, 3-row ring, nt-load(unshifted planes) nt-store waves>=5", 2, 16},
                                // 9, 14, 15 and 10 with tiles in XCD-banded order
                                {64, 1, "batch two steps per launch, 64x16 tiles, 3-row ring, nt-load(unshifted planes) nt-store, XCD-banded", 2, 16},
                                {256, 1, "batch two steps per launch, 256x16 tiles, 3-row ring, nt-load(unshifted planes) nt-store, XCD-banded", 2, 16},
                                {256, 1, "batch two steps per launch, 256x16 tiles, split rings, nt-load(unshifted planes) nt-store, XCD-banded", 2, 16},
                                {64, 1, "batch two steps per launch, 64x16 tiles, split rings, nt-load(unshifted planes) nt-store, XCD-banded", 2, 16},
                                {128, 1, "batch two steps per launch, 128x16 tiles, 3-row ring, nt-load(unshifted planes) nt-store", 2, 16},
                                {128, 1, "batch two steps per launch, 128x16 tiles, split rings, nt-load(unshifted planes) nt-store", 2, 16},
                                // register pipelines (every collision rule): blk = 64 - 2 (steps - 1) columns
                                {62, 1, "batch register pipeline, 2 steps per launch, 62x8 tiles", 2, 8},
                                {62, 1, "batch register pipeline, 2 steps per launch, 62x16 tiles", 2, 16},
                                {62, 1, "batch register pipeline, 2 steps per launch, 62x32 tiles", 2, 32},
                                {60, 1, "batch register pipeline, 3 steps per launch, 60x16 tiles", 3, 16},
                                {60, 1, "batch register pipeline, 3 steps per launch, 60x32 tiles", 3, 32},
                                {58, 1, "batch register pipeline, 4 steps per launch, 58x16 tiles", 4, 16},
                                {58, 1, "batch register pipeline, 4 steps per launch, 58x32 tiles", 4, 32}};
// Single-step batch shapes (every collision rule), then two-step shapes of
// MinxEnt4, then register pipelines (every rule).
constexpr int kNumB9One = 9;
constexpr int kNumB9Pipes = 7;
constexpr int kNumB9 = sizeof(kShapesB9) / sizeof(kShapesB9[0]);
constexpr int kFirstB9Pipe = kNumB9 - kNumB9Pipes;

// Entry of kShapesB9 of shape v of a collision rule, or -1.
int shape_of_b9(int coll, int v)
{
    if (v < 0) return -1;
    if (coll != CO_MINXENT4 && v >= kNumB9One) v += kFirstB9Pipe - kNumB9One;
    return v < kNumB9 ? v : -1;
}
constexpr ShapeB kShapesB3[] = {{256, 1, "batch 256x1 nodes/block"}, {128, 1, "batch 128x1 nodes/block"},
                                {256, 4, "batch 256x4 nodes/block"}, {256, 8, "batch 256x8 nodes/block"},
                                {256, 4, "batch 256x4 nodes/block nt-load nt-store"},
                                {256, 8, "batch 256 groups of 8 nodes, 16-byte vectors"},
                                {256, 8, "batch 256 groups of 8 nodes, 16-byte vectors nt-load nt-store"},
                                {128, 8, "batch 128 groups of 8 nodes, 16-byte vectors nt-load nt-store"},
                                {128, 1, "batch 128x1 nodes/block, XCD-banded"},
                                {256, 8, "batch 256 groups of 8 nodes, 16-byte vectors, XCD-banded"},
                                // blk: nodes of a tile, 64 per lane and node less the 64 of the ends
                                {64, 1, "batch nodes in registers, 2 per lane, up to 32 steps per launch", 32},
                                {192, 1, "batch nodes in registers, 4 per lane, up to 32 steps per launch", 32},
                                {448, 1, "batch nodes in registers, 8 per lane, up to 32 steps per launch", 32}};
constexpr int kFirstRegsB3 = 10;

template <int ST>
hipError_t dispatch3b(int v, const void *src, void *dst, const StepArgs &a_in, hipStream_t s)
{
    using T = typename Form<ST>::T;
    // Tiles run in launch order; shapes 8 and 9 are 1 and 5 with tiles in
    // XCD-banded order instead (measured slower, kept as candidates); 10 on
    // take several steps per launch.
    StepArgs a = a_in;
    a.xcd_swizzle = 0;
    if (v >= kFirstRegsB3) return launch_d1q3_regs(ST, 2 << (v - kFirstRegsB3), 1, src, dst, a, s);
    if (v >= 8) {
        a.xcd_swizzle = 1;
        v = v == 8 ? 1 : 5;
    }
    switch (v) {
    case 0: hipLaunchKernelGGL((k_d1q3_batch<ST, 256, 1>), dim3(a.ntiles), dim3(256), 0, s, (const T *)src, (T *)dst, a); break;
    case 1: hipLaunchKernelGGL((k_d1q3_batch<ST, 128, 1>), dim3(a.ntiles), dim3(128), 0, s, (const T *)src, (T *)dst, a); break;
    case 2: hipLaunchKernelGGL((k_d1q3_batch<ST, 256, 4>), dim3(a.ntiles), dim3(256), 0, s, (const T *)src, (T *)dst, a); break;
    case 3: hipLaunchKernelGGL((k_d1q3_batch<ST, 256, 8>), dim3(a.ntiles), dim3(256), 0, s, (const T *)src, (T *)dst, a); break;
    case 4: hipLaunchKernelGGL((k_d1q3_batch<ST, 256, 4, 3>), dim3(a.ntiles), dim3(256), 0, s, (const T *)src, (T *)dst, a); break;
    case 5: hipLaunchKernelGGL((k_d1q3_batch_v8<ST, 256>), dim3(a.ntiles), dim3(256), 0, s, (const T *)src, (T *)dst, a); break;
    case 6: hipLaunchKernelGGL((k_d1q3_batch_v8<ST, 256, 3>), dim3(a.ntiles), dim3(256), 0, s, (const T *)src, (T *)dst, a); break;
    case 7: hipLaunchKernelGGL((k_d1q3_batch_v8<ST, 128, 3>), dim3(a.ntiles), dim3(128), 0, s, (const T *)src, (T *)dst, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int ST>
hipError_t init_st(int lattice, const NodeRange &r, const double *rho, const double *ux, const double *uy,
                   const double *f, void *buf, float scale, hipStream_t s)
{
    using T = typename Form<ST>::T;
    const unsigned blocks = (unsigned)((r.g1 - r.g0 + 255) / 256);
#define LBM_INIT(B, BATCH) \
    hipLaunchKernelGGL((k_init<ST, B, BATCH>), dim3(blocks), dim3(256), 0, s, r, rho, ux, uy, f, (T *)buf, scale)
    if (lattice == 9) {
        if (r.inst) LBM_INIT(9, true);
        else LBM_INIT(9, false);
    } else {
        if (r.inst) LBM_INIT(3, true);
        else LBM_INIT(3, false);
    }
#undef LBM_INIT
    return hipGetLastError();
}

template <int ST>
hipError_t gather_st(int lattice, const NodeRange &r, const void *buf, double *rho, double *ux, double *uy,
                     double *f, int64_t fstride, float iscale, hipStream_t s)
{
    using T = typename Form<ST>::T;
    const unsigned blocks = (unsigned)((r.g1 - r.g0 + 255) / 256);
    if (lattice == 9)
        hipLaunchKernelGGL((k_gather<ST, 9>), dim3(blocks), dim3(256), 0, s, r, (const T *)buf, rho, ux, uy, f, fstride,
                           iscale);
    else
        hipLaunchKernelGGL((k_gather<ST, 3>), dim3(blocks), dim3(256), 0, s, r, (const T *)buf, rho, ux, uy, f, fstride,
                           iscale);
    return hipGetLastError();
}

}  // namespace

int d2q9_variant_count(int coll) { return coll == CO_MINXENT4 ? kNumShapes : kNumOneOther + kNumWindows + kNumPipes; }
int d2q9_variant_steps(int coll, int v)
{
    const int k = shape_of(coll, v);
    return k >= 0 ? kShapes[k].steps : 1;
}
bool d2q9_variant_window(int coll, int v)
{
    const int k = shape_of(coll, v);
    return k >= kFirstWindow && k < kFirstPipe;
}

// The longer of two times that overlap, a little more where they are close.
static double soft_max(double a, double b) { return std::sqrt(std::sqrt(a * a * a * a + b * b * b * b)); }

// One-step launches cost 4.4 us each and 18 ps per node (FP64 MinxEnt; 5-17 in
// the others), and the bytes of a step at 6.2 TB/s beyond the caches (FP64,
// us per step: 6.2, 8.4, 10.7, 24, 55 and 110 at 257^2, 400^2, 600^2, 1000^2,
// 1400^2 and 2048^2).  The window shapes take 1.5 us per step at 32^2, 1.8 at
// 128^2, 3.4 at 257^2 and 6.3 at 480^2, so they lead up to about 550^2; the
// register pipelines lead from there on (FP64 MinxEnt4 / MRT, us per step:
// 1000^2 18.8 / 12.0, 2048^2 60 / 50, 4096^2 221 / 157, against 24 / 24, 110 / 109
// and 430 / 432 for one step per launch).
int d2q9_default_variant(int st, int coll, int nx, int ny, int bc)
{
    const int windows = d2q9_variant_count(coll) - kNumPipes - kNumWindows;
    const bool newton = coll == CO_MINXENT4 || coll == CO_MINXENT2;
    const double nodes = (double)nx * ny, elem = st == ST_F64 ? 8 : (st == ST_F16DEV ? 2 : 4);
    const double node_ps[2][4] = {{16.7, 8.8, 8.2, 5.4}, {18.4, 8.5, 9.7, 6.6}};
    double best = soft_max(4.6 + node_ps[newton][st] * 1e-6 * nodes, nodes * 18 * elem / 6.2e6);
    int v = 0;
    int steps[kNumWindows];
    for (int k = 0; k < kNumWindows; ++k) steps[k] = kShapes[kFirstWindow + k].steps;
    WindowTile tile;
    const int window = d2q9_window_best(st, coll, nx, ny, bc, steps, kNumWindows, best, &tile, &best);
    if (window >= 0) v = windows + window;
    // The shapes whose rows go by the lattice; more steps only if they gain more
    // than the estimates are off by (600^2 FP64: 9.5 us with two, 10.1 with three).
    for (int k = 0; k < 3; ++k) {
        double us = 0;
        if (d2q9_pipe_rows(st, coll, nx, ny, kShapes[kFirstPipe + k].steps, &us, 0.95 * best)) {
            best = us;
            v = windows + kNumWindows + k;
        }
    }
    return v;
}

hipError_t prepare_d2q9_variant(int st, int coll, int v)
{
    if (shape_of(coll, v) >= kFirstWindow || d2q9_variant_steps(coll, v) != 2) return hipSuccess;
    const StepArgs none{};
    switch (st) {
    case ST_F64: return dispatch9t2<ST_F64, CO_MINXENT4>(v, true, nullptr, nullptr, none, nullptr);
    case ST_F32N64: return dispatch9t2<ST_F32N64, CO_MINXENT4>(v, true, nullptr, nullptr, none, nullptr);
    case ST_F32: return dispatch9t2<ST_F32, CO_MINXENT4>(v, true, nullptr, nullptr, none, nullptr);
    case ST_F16DEV: return dispatch9t2<ST_F16DEV, CO_MINXENT4>(v, true, nullptr, nullptr, none, nullptr);
    default: return hipErrorInvalidValue;
    }
}
const char *d2q9_variant_name(int coll, int v)
{
    const int k = shape_of(coll, v);
    return k >= 0 ? kShapes[k].name : "?";
}
int d1q3_variant_count() { return kNumShapes3; }
const char *d1q3_variant_name(int v) { return (v >= 0 && v < kNumShapes3) ? kShapes3[v].name : "?"; }
constexpr int kNumB3 = sizeof(kShapesB3) / sizeof(kShapesB3[0]);
int batch_variant_count(int lattice, int coll)
{
    if (lattice == 3) return kNumB3;
    return coll == CO_MINXENT4 ? kNumB9 : kNumB9One + kNumB9Pipes;
}
int batch_variant_steps(int lattice, int coll, int v)
{
    if (lattice == 3) return (v >= 0 && v < kNumB3) ? kShapesB3[v].steps : 1;
    const int k = shape_of_b9(coll, v);
    return k >= 0 ? kShapesB9[k].steps : 1;
}
// A launch of one step gains nothing from rows or nodes in registers and computes
// the windows' overlaps (128 cavities of 32^2 to 512^2, us, register pipeline /
// shape 0: FP32 270 / 194, FP64 468 / 345).
int batch_one_step(int lattice, int coll, int v)
{
    return (lattice == 3 ? v >= kFirstRegsB3 : shape_of_b9(coll, v) >= kFirstB9Pipe) ? 0 : v;
}
int d1q3_variant_steps(int v) { return (v >= 0 && v < kNumShapes3) ? kShapes3[v].steps : 1; }

// Us per step of a single lattice, FP64: 0.33 to 0.35 at 800 to 50000 nodes with
// 2 nodes per lane; 0.74 / 0.78 / 0.95 with 2 / 4 / 8 at 200000; 2.29 / 1.83 / 2.01
// at a million; batches of 8 and 63 million nodes run fastest with 8 (one step per
// launch: 3.7 us up to 200000 nodes, 8.6 at a million).
int d1q3_default_variant(int batch, int64_t nodes)
{
    const int i = nodes < 400000 ? 0 : (nodes < 3000000 ? 1 : 2);  // 2, 4 or 8 nodes per lane
    return (batch ? kFirstRegsB3 : kFirstRegs3) + i;
}
int batch_tile_nodes(int lattice, int coll, int v)
{
    if (lattice == 3) return (v >= 0 && v < kNumB3) ? kShapesB3[v].blk * kShapesB3[v].npt : 0;
    const int k = shape_of_b9(coll, v);
    if (k < 0) return 0;
    if (kShapesB9[k].rows) return -(kShapesB9[k].blk * 4096 + kShapesB9[k].rows);
    return kShapesB9[k].blk * kShapesB9[k].npt;
}

hipError_t prepare_batch_variant(int st, int coll, int v)
{
    if (coll != CO_MINXENT4 || v < kNumB9One || v >= kFirstB9Pipe) return hipSuccess;
    const StepArgs none{};
    switch (st) {
    case ST_F64: return dispatch9bt2<ST_F64, CO_MINXENT4>(v, true, nullptr, nullptr, none, nullptr);
    case ST_F32N64: return dispatch9bt2<ST_F32N64, CO_MINXENT4>(v, true, nullptr, nullptr, none, nullptr);
    case ST_F32: return dispatch9bt2<ST_F32, CO_MINXENT4>(v, true, nullptr, nullptr, none, nullptr);
    case ST_F16DEV: return dispatch9bt2<ST_F16DEV, CO_MINXENT4>(v, true, nullptr, nullptr, none, nullptr);
    default: return hipErrorInvalidValue;
    }
}
const char *batch_variant_name(int lattice, int coll, int v)
{
    if (lattice == 3) return (v >= 0 && v < kNumB3) ? kShapesB3[v].name : "?";
    const int k = shape_of_b9(coll, v);
    return k >= 0 ? kShapesB9[k].name : "?";
}

bool d2q9_variant_pipe(int coll, int v) { return shape_of(coll, v) >= kFirstPipe; }
int d2q9_variant_rows(int coll, int v)
{
    const int k = shape_of(coll, v);
    return k >= kFirstPipe ? kShapes[k].by : 0;
}

// Waves per SIMD that the registers of a register pipeline allow.
static int pipe_waves(int st, int coll, int k)
{
    const bool newton = coll == CO_MINXENT4 || coll == CO_MINXENT2;
    return st == ST_F64 ? (newton ? 6 - k : 7 - k) : (st == ST_F32N64 && newton ? 4 : 6);
}

// Microseconds of one collision of a wave of a register pipeline: its latency,
// and its issue.  Fitted with the fixed time and the rate of d2q9_pipe_rows to
// 7,200 launches (60,000 nodes to 3500^2, 4 to 32 rows, every rule and form; off
// by 5-9% rms).
static double pipe_latency_us(int st, int coll)
{
    const double us[2][4] = {{0.65, 0.54, 0.55, 0.56}, {1.08, 0.98, 0.85, 0.89}};
    return us[coll == CO_MINXENT4 || coll == CO_MINXENT2][st];
}
static double pipe_issue_us(int st, int coll)
{
    const double us[2][4] = {{0.40, 0.32, 0.22, 0.29}, {0.68, 0.63, 0.40, 0.45}};
    return us[coll == CO_MINXENT4 || coll == CO_MINXENT2][st];
}

int d2q9_pipe_rows(int st, int coll, int nx, int ny, int k, double *us_per_step, double below)
{
    const int occ = pipe_waves(st, coll, k);
    const double latency = pipe_latency_us(st, coll), issue = pipe_issue_us(st, coll);
    const double elem = st == ST_F64 ? 8 : (st == ST_F16DEV ? 2 : 4);
    const int w = 64 - 2 * (k - 1);
    const int strips = (nx + w - 1) / w;
    const double bytes = (double)nx * ny * 9 * elem;
    double best = below * k;
    int rows = 0;
    for (int h = 1; h <= 48; ++h) {
        if (h > ny) break;
        const int collisions = k * h + k * (k - 1);  // of one wave
        if (4.8 + collisions * latency >= best) break;  // more rows take longer
        const int blocks = (strips * ((ny + h - 1) / h) + 3) / 4;
        // Blocks per compute unit: whole while all are resident at once; on
        // average, and in FP64 half a block of tail, when they come and go.
        const int whole = (blocks + kWindowCus - 1) / kWindowCus;
        const double r = whole <= occ ? whole : (double)blocks / kWindowCus + (st == ST_F64 ? 0.55 : 0.0);
        const double memory = bytes * (2.1 + 0.6 * k / h) / 5.2e6;
        if (4.8 + std::max(collisions * r * issue, memory) >= best) continue;
        const double compute = collisions * soft_max(latency, r * issue);
        const double us = 4.8 + soft_max(compute, memory);
        if (us < best) {
            best = us;
            rows = h;
        }
    }
    if (us_per_step) *us_per_step = rows ? best / k : 1e30;
    return rows;
}

// One step per launch or a register pipeline, by the estimates of both: which
// one is faster turns on how full the tiles are.  A wave of a pipeline takes all
// its rows and the k - 1 around them one after another, 64 columns wide whatever
// the lattice holds, and a block of 256 nodes one collision.  Measured us per
// step, one step per launch / pipeline of three (FP32) or two (FP16 deviations):
// 1000 cavities of 100^2 FP32 227 / 108, 1100 of 17^2 11.5 / 22.6, 600 of 64^2 28.9 /
// 40.4, 50 of 4 x 800 12.1 / 28.7, 1000 of them 513 / 327; 600 of 64^2 FP16 deviations
// 24.0 / 41.7, 1000 of 100^2 128 / 107.  Three steps lead in FP64 and FP32 and two in
// the other forms, which are bound by issue (128 cavities, 5.2 million nodes,
// MLUPS, one step per launch / two-step rings / pipeline of two steps / of three:
// FP64 35,700 / 49,500 / 45,700 / 56,100, FP32 71,000 / 84,300 / 88,300 / 94,700,
// FP32 storage / FP64 compute 63,500 / 58,700 / 72,000 / 66,300, SRT FP32 69,000 / - /
// 93,600 / 124,000).   The estimates are off by
// 16-21% rms over 340 batches of 8 thousand to 12 million nodes, lattices of 3 to
// 1000 columns, every rule and form, so the pipeline has to lead by 15%.  The time
// is then 0.90 of that of one step per launch on average and at most 1.14 of it
// (1.04 and 3.7 with a pipeline wherever the tiles make 2048 waves).
int batch_default_variant(int st, int coll, const Inst *inst, int n)
{
    const bool newton = coll == CO_MINXENT4 || coll == CO_MINXENT2;
    const int k = st == ST_F64 || st == ST_F32 ? 3 : 2;
    const int v = batch_variant_count(9, coll) - kNumB9Pipes + (k == 3 ? 3 : 1);
    const int w = 64 - 2 * (k - 1), rows = kShapesB9[shape_of_b9(coll, v)].rows;
    const double elem = st == ST_F64 ? 8 : (st == ST_F16DEV ? 2 : 4);
    double nodes = 0, blocks = 0;  // of one step per launch
    double bytes = 0, narrow = 0;  // lines of a plane; of them, in rows of 32 bytes and less
    double tiles = 0, collisions = 0;
    int tallest = 0;
    for (int i = 0; i < n; ++i) {
        const double nx = inst[i].nx, ny = inst[i].ny;
        const double row = std::ceil(nx * elem / 128), strips = std::ceil(nx / w), t = std::ceil(ny / rows);
        nodes += nx * ny;
        blocks += std::ceil(nx * ny / 256);
        bytes += ny * row * 128;
        narrow += nx * elem <= 32 ? ny * row * 128 : 0;
        tiles += strips * t;
        collisions += strips * (k * ny + t * k * (k - 1));
        tallest = std::max(tallest, std::min(inst[i].ny, rows));
    }
    const double node_ps[2][4] = {{16.7, 8.8, 8.2, 5.4}, {18.4, 8.5, 9.7, 6.6}};
    // Bytes at the rate of what the caches hold, or of memory (narrow rows, whose
    // stores fill sectors in part, at 3.6 TB/s).
    const double moved = 18 * bytes < 350e6 ? 18 * bytes / 7.6e6 : 18 * (bytes + 0.4 * narrow) / 5.0e6;
    const double issue = pipe_issue_us(st, coll);
    const double one = soft_max(4.6 + std::max(node_ps[newton][st] * 1e-6 * nodes, blocks / kWindowCus * issue), moved);
    const double mean = tiles / 4 / kWindowCus, whole = std::ceil(mean);
    const double r = whole <= pipe_waves(st, coll, k) ? whole : mean + (st == ST_F64 ? 0.55 : 0.0);
    const double longest = k * tallest + k * (k - 1);
    const double compute = soft_max(longest * pipe_latency_us(st, coll), collisions / tiles * r * issue);
    const double pipe = (4.8 + soft_max(compute, 9 * bytes * (2.1 + 0.6 * k / tallest) / 5.2e6)) / k;
    return pipe < 0.85 * one ? v : 0;
}

namespace {
hipError_t launch_d2q9_pipe(int st, int coll, int k, int batch, const void *src, void *dst, const StepArgs &a_in,
                            hipStream_t s)
{
    StepArgs a = a_in;
    if (a.tile_rows < 1) return hipErrorInvalidValue;
    if (!batch) {
        const int w = 64 - 2 * (k - 1);
        a.tiles_x = (a.one.nx + w - 1) / w;
        const int rows = (a.one.ny + a.tile_rows - 1) / a.tile_rows;  // of tiles
        a.tall = rows;
        a.low_rows = a.tile_rows;
        const int64_t held = (int64_t)kWindowCus * 4 * pipe_waves(st, coll, k);
        const bool newton = coll == CO_MINXENT4 || coll == CO_MINXENT2;
        // Where the waves come and go, a quarter of those held at once take half
        // the rows and run last, so that the chip empties in half the time; the
        // rows they take twice cost less than that (us per step, one height /
        // two: headline form 4096^2 179.8 / 175.2, FP64 223.4 / 220.1, FP16 deviations
        // 3001 x 2203 51.2 / 48.9; half of the waves held, or a quarter of the rows:
        // 1-2% slower).  Not for the other rules, which the memory bounds
        // (SRT FP64 4096^2 151.8 / 151.6 to 155.7).
        if (newton && (int64_t)a.tiles_x * rows > held && a.tile_rows >= 8) {
            a.tall = std::max(0, rows - (int)((held / 4 + a.tiles_x / 2) / a.tiles_x));
            a.low_rows = a.tile_rows / 2;
        }
        const int below = a.tall * a.tile_rows;
        const int64_t tiles =
            (int64_t)a.tiles_x * (a.tall + (std::max(0, a.one.ny - below) + a.low_rows - 1) / a.low_rows);
        if (tiles > 0x7fffffff) return hipErrorInvalidValue;
        a.ntiles = (int32_t)tiles;
    }
    switch (coll) {
    case CO_MINXENT4: return launch_d2q9_pipe_0(st, k, batch, src, dst, a, s);
    case CO_MINXENT2: return launch_d2q9_pipe_1(st, k, batch, src, dst, a, s);
    case CO_SRT: return launch_d2q9_pipe_2(st, k, batch, src, dst, a, s);
    case CO_TRT: return launch_d2q9_pipe_3(st, k, batch, src, dst, a, s);
    case CO_MRT: return launch_d2q9_pipe_4(st, k, batch, src, dst, a, s);
    default: return hipErrorInvalidValue;
    }
}
}  // namespace

hipError_t launch_d2q9_step(int st, int coll, int v, const void *src, void *dst, const StepArgs &a, hipStream_t s)
{
    if (v < 0 || v >= d2q9_variant_count(coll)) return hipErrorInvalidValue;
    const int k = shape_of(coll, v);
    // A launch of one step runs shape 0: no lattice is too tall or too large for
    // it, and it is the faster one (us, shape 0 / a window of one step: 257^2 FP64
    // 6.5 / 7.9, SRT FP32 5.0 / 7.2; 400^2 FP16 deviations 5.8 / 8.7; 17^2 4.8 / 5.2).
    if (k >= kFirstWindow && a.max_steps <= 1) v = 0;
    else if (k >= kFirstPipe) return launch_d2q9_pipe(st, coll, a.max_steps, 0, src, dst, a, s);
    else if (k >= kFirstWindow) return launch_d2q9_window(st, coll, src, dst, a, s);
    switch (st) {
    case ST_F64: return dispatch9c<ST_F64>(coll, v, src, dst, a, s);
    case ST_F32N64: return dispatch9c<ST_F32N64>(coll, v, src, dst, a, s);
    case ST_F32: return dispatch9c<ST_F32>(coll, v, src, dst, a, s);
    case ST_F16DEV: return dispatch9c<ST_F16DEV>(coll, v, src, dst, a, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_d2q9_batch_step(int st, int coll, int v, const void *src, void *dst, const StepArgs &a,
                                  hipStream_t s)
{
    v = shape_of_b9(coll, v);
    if (v < 0) return hipErrorInvalidValue;
    if (v >= kFirstB9Pipe) {
        StepArgs p = a;
        p.tile_rows = kShapesB9[v].rows;
        return launch_d2q9_pipe(st, coll, kShapesB9[v].steps, 1, src, dst, p, s);
    }
    switch (st) {
    case ST_F64: return dispatch9bc<ST_F64>(coll, v, src, dst, a, s);
    case ST_F32N64: return dispatch9bc<ST_F32N64>(coll, v, src, dst, a, s);
    case ST_F32: return dispatch9bc<ST_F32>(coll, v, src, dst, a, s);
    case ST_F16DEV: return dispatch9bc<ST_F16DEV>(coll, v, src, dst, a, s);
    default: return hipErrorInvalidValue;
    }
}

namespace {
template <int ST, int CO>
hipError_t lds_go(const void *src, void *dst, const StepArgs &a, int nsteps, int block, size_t smem, hipStream_t s)
{
    using T = typename Form<ST>::T;
    hipError_t e = hipFuncSetAttribute((const void *)k_d2q9_lds<ST, CO>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                       (int)smem);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_d2q9_lds<ST, CO>), dim3(a.ntiles), dim3(block), smem, s, (const T *)src, (T *)dst, a,
                       nsteps);
    return hipGetLastError();
}

template <int ST>
hipError_t lds_coll(int coll, const void *src, void *dst, const StepArgs &a, int nsteps, int block, size_t smem,
                    hipStream_t s)
{
    switch (coll) {
    case CO_MINXENT4: return lds_go<ST, CO_MINXENT4>(src, dst, a, nsteps, block, smem, s);
    case CO_MINXENT2: return lds_go<ST, CO_MINXENT2>(src, dst, a, nsteps, block, smem, s);
    case CO_SRT: return lds_go<ST, CO_SRT>(src, dst, a, nsteps, block, smem, s);
    case CO_TRT: return lds_go<ST, CO_TRT>(src, dst, a, nsteps, block, smem, s);
    case CO_MRT: return lds_go<ST, CO_MRT>(src, dst, a, nsteps, block, smem, s);
    default: return hipErrorInvalidValue;
    }
}
}  // namespace

hipError_t launch_d2q9_lds(int st, int coll, const void *src, void *dst, const StepArgs &a, int nsteps, int block,
                           size_t smem, hipStream_t s)
{
    if (nsteps <= 0) return hipSuccess;
    switch (st) {
    case ST_F64: return lds_coll<ST_F64>(coll, src, dst, a, nsteps, block, smem, s);
    case ST_F32N64: return lds_coll<ST_F32N64>(coll, src, dst, a, nsteps, block, smem, s);
    case ST_F32: return lds_coll<ST_F32>(coll, src, dst, a, nsteps, block, smem, s);
    case ST_F16DEV: return lds_coll<ST_F16DEV>(coll, src, dst, a, nsteps, block, smem, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_d1q3_step(int st, int v, const void *src, void *dst, const StepArgs &a, hipStream_t s)
{
    // A launch of one step gains nothing from nodes in registers, and loads the
    // windows' overlaps (us, in registers / shape 0: a million nodes FP64 15.6 / 9.1,
    // ten million 361 / 84).
    if (v >= kFirstRegs3 && a.max_steps <= 1) v = 0;
    switch (st) {
    case ST_F64: return dispatch3<ST_F64>(v, src, dst, a, s);
    case ST_F32N64: return dispatch3<ST_F32N64>(v, src, dst, a, s);
    case ST_F32: return dispatch3<ST_F32>(v, src, dst, a, s);
    case ST_F16DEV: return dispatch3<ST_F16DEV>(v, src, dst, a, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_d1q3_batch_step(int st, int v, const void *src, void *dst, const StepArgs &a, hipStream_t s)
{
    if (v < 0 || v >= batch_variant_count(3, 0)) return hipErrorInvalidValue;
    switch (st) {
    case ST_F64: return dispatch3b<ST_F64>(v, src, dst, a, s);
    case ST_F32N64: return dispatch3b<ST_F32N64>(v, src, dst, a, s);
    case ST_F32: return dispatch3b<ST_F32>(v, src, dst, a, s);
    case ST_F16DEV: return dispatch3b<ST_F16DEV>(v, src, dst, a, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_init(int lattice, int st, const NodeRange &r, const double *rho, const double *ux, const double *uy,
                       const double *f, void *buf, float scale, hipStream_t s)
{
    if (r.g1 <= r.g0) return hipSuccess;
    switch (st) {
    case ST_F64: return init_st<ST_F64>(lattice, r, rho, ux, uy, f, buf, scale, s);
    case ST_F32N64: return init_st<ST_F32N64>(lattice, r, rho, ux, uy, f, buf, scale, s);
    case ST_F32: return init_st<ST_F32>(lattice, r, rho, ux, uy, f, buf, scale, s);
    case ST_F16DEV: return init_st<ST_F16DEV>(lattice, r, rho, ux, uy, f, buf, scale, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_gather(int lattice, int st, const NodeRange &r, const void *buf, double *rho, double *ux, double *uy,
                         double *f, int64_t fstride, float iscale, hipStream_t s)
{
    if (r.g1 <= r.g0) return hipSuccess;
    switch (st) {
    case ST_F64: return gather_st<ST_F64>(lattice, r, buf, rho, ux, uy, f, fstride, iscale, s);
    case ST_F32N64: return gather_st<ST_F32N64>(lattice, r, buf, rho, ux, uy, f, fstride, iscale, s);
    case ST_F32: return gather_st<ST_F32>(lattice, r, buf, rho, ux, uy, f, fstride, iscale, s);
    case ST_F16DEV: return gather_st<ST_F16DEV>(lattice, r, buf, rho, ux, uy, f, fstride, iscale, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_copy(void *dst, const void *src, size_t bytes, hipStream_t s)
{
    const size_t n = bytes / 16;
    if (n == 0) return hipSuccess;
    const size_t blocks = (n + 256 * kCopyVec - 1) / (256 * kCopyVec);
    if (blocks > 0x7fffffffu) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_copy, dim3((unsigned)blocks), dim3(256), 0, s, (u32x4 *)dst, (const u32x4 *)src, n);
    return hipGetLastError();
}

hipError_t launch_add_step_base(int64_t *b, int64_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_step_base, dim3(1), dim3(64), 0, s, b, n, 1);
    return hipGetLastError();
}

hipError_t launch_set_step_base(int64_t *b, int64_t v, hipStream_t s)
{
    hipLaunchKernelGGL(k_step_base, dim3(1), dim3(64), 0, s, b, v, 0);
    return hipGetLastError();
}

hipError_t launch_clear_status(DevStatus *st, int n, hipStream_t s)
{
    hipLaunchKernelGGL(k_clear_status, dim3((n + 255) / 256), dim3(256), 0, s, st, n);
    return hipGetLastError();
}

}  // namespace lbm
