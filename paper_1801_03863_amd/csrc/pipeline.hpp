// pipeline.hpp -- D2Q9, one lattice or a batch, K steps per launch with everything
// between the first pull and the last store in registers.
//
// A wave owns an output tile of 64 - 2 (K - 1) columns and H rows, and walks
// up a window that is K - 1 nodes wider on every side, one row per iteration:
// its 64 lanes are 64 neighbouring columns.  In each iteration stage 1 computes the next
// window row straight from the other buffer, as a single-step launch does;
// stage s computes the row s - 1 below it, one step later, from what stage
// s - 1 left in registers; stage K stores.  A stage needs of the one before
// it planes 4, 7, 8 of the row just computed, 0, 1, 3 of the row before and 2,
// 5, 6 of the row before that, so nine values per lane (three more at a top
// wall) carry a stage from row to row; the six that move sideways pass to
// the neighbouring lane by a wave shift.  No LDS and no barrier: waves never
// wait for each other.  Every value is rounded to the storage type after
// every step and every node is computed with the same arithmetic, so results
// are bitwise equal to single steps.
//
// At lattice ends that do not wrap the window is cut (rows) or its lanes
// beyond the end are dead (columns), and the end nodes pull from themselves;
// on axes that wrap the window runs on through the other end.
//
// What bounds it: VALU issue for the Newton rules (FP64 needs 153 registers at
// three steps, 3 waves per SIMD), memory for the relaxation rules.  K trades
// bytes (one read and one write of every population per K steps) against lanes and
// rows computed twice (64 / (64 - 2 (K - 1)) and (H + K - 1) / H on average).  The ring
// of rows in LDS of k_d2q9_t2 holds two steps only, and its waves wait for
// each other at every row.  Measured on the 4096^2 cavity, us per step, best
// shape before -> here: FP64 250 -> 221, FP32 storage / FP64 compute 187 -> 178,
// FP32 129 -> 119, FP16 deviations 119.5 -> 115.5, MRT FP64 432 -> 157, SRT FP32
// 213 -> 82; 2048^2 FP64 74 -> 61-65; 1000^2 MRT FP64 24.2 -> 15.0.  Batches, MLUPS:
// 512 cavities FP32 103,500 -> 118,000, FP64 57,000 -> 63,000; 128 cavities SRT FP32
// 69,000 -> 147,000, MRT FP64 35,700 -> 61,000.
#pragma once

#include <type_traits>

#include "device.hpp"

namespace lbm {

// What a stage keeps of its output for the next one (after the sideways
// move): a = row last computed, b = the row before.
template <class T>
struct StageRows {
    T a0, a1, a3;
    T a2, a5, a6, b2, b5, b6;
    T a4, a7, a8;  // read again only at a top wall
};

template <int ST, int CO, int K, bool BATCH>
__global__ __launch_bounds__(256) void k_d2q9_rp(const typename Form<ST>::T *__restrict__ src_all,
                                                 typename Form<ST>::T *__restrict__ dst_all, StepArgs a)
{
    using C = typename Form<ST>::C;
    using T = typename Form<ST>::T;
    constexpr int W = 64 - 2 * (K - 1);  // columns of a tile
    // Adjacent tiles share lines: each XCD takes a band of the tall tiles, then
    // one of the low ones.
    int b = (int)blockIdx.x;
    if constexpr (BATCH) {
        b = xcd_remap(b, (int)gridDim.x);
    } else {
        const int t = a.tall * a.tiles_x / 4, n = (int)gridDim.x;
        b = b < t ? xcd_remap(b, t) : t + xcd_remap(b - t, n - t);
    }
    const int entry = b * 4 + __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    if (entry >= a.ntiles) return;  // wave-uniform
    // A batch's tile table gives the instance and the tile within it.
    const int ii = BATCH ? a.tile_inst[entry] : 0;
    const int tile = BATCH ? a.tile_first[entry] : entry;
    const Inst &lat = BATCH ? a.inst[ii] : a.one;
    Inst in;  // what the collision reads, held in registers
    in.omega = lat.omega;
    in.omega2 = lat.omega2;
    in.rho0 = lat.rho0;
    const int nx = lat.nx, ny = lat.ny, pitch = lat.pitch;
    const int64_t P = lat.plane;
    const T *src = src_all + (BATCH ? lat.offset : 0);
    T *dst = dst_all + (BATCH ? lat.offset : 0);
    const int bc = a.bc;
    const bool xw = bc == BC_PERIODIC;
    const bool yw = bc == BC_PERIODIC || bc == BC_TUBE;
    const bool cavity = bc == BC_CAVITY;
    const int tiles_x = BATCH ? (nx + W - 1) / W : a.tiles_x;
    const int ty = tile / tiles_x, tx = tile - ty * tiles_x;
    const bool low = !BATCH && ty >= a.tall;
    const int H = low ? a.low_rows : a.tile_rows;
    const int lane = (int)(threadIdx.x & 63);
    const int x = tx * W - (K - 1) + lane, y0 = low ? a.tall * a.tile_rows + (ty - a.tall) * H : ty * H;
    const int yn = min(ny, y0 + H);  // own rows [y0, yn)
    const bool own_x = lane >= K - 1 && lane < 64 - (K - 1) && x < nx;
    // Steps this wave takes (wave-uniform): K, or in a batch fewer for a launch
    // of fewer steps or an instance that reaches its step limit, none for one
    // that has (it carries its nodes over).
    int kdo = K;
    if constexpr (BATCH) {
        const int64_t s0 = a.step + (a.step_base ? *a.step_base : 0);
        kdo = (int)max((int64_t)0, min((int64_t)min(K, a.max_steps), lat.stop - s0));
        if (kdo <= 0) {
            if (own_x)
                for (int y = y0; y < yn; ++y) carry_node(src, dst, P, 9, y * pitch + x);
            return;
        }
    }
    int xs = x;  // lattice column of this lane
    if (xw) {
        if (xs < 0) xs += nx;
        if (xs >= nx) xs -= nx;
        if ((unsigned)xs >= (unsigned)nx) xs = ((xs % nx) + nx) % nx;
    } else {
        xs = min(max(xs, 0), nx - 1);
    }
    const bool edge = tx == 0 || tx * W + 64 - (K - 1) >= nx;  // wave-uniform: a lane at or beyond a lattice end
    const bool at_left = !xw && x == 0, at_right = !xw && x == nx - 1;
    const Cols cols = columns(xs, edge, nx, bc, sizeof(T));
    C ref[9];
    ref9<C>(C(in.rho0), ref);

    int bad[K];
#pragma unroll
    for (int s = 0; s < K; ++s) bad[s] = kNoNode;
    int guarded = 0;

    // The walk up the window.  INNER: the window and the rows and columns it
    // pulls from lie inside the lattice and hold no wall or lid node, which is
    // known for the whole wave, so that copy carries no wall, wrap or lid code
    // (about a twentieth of the vector instructions).
    auto walk = [&](auto inner) __attribute__((always_inline)) {
        constexpr bool INNER = decltype(inner)::value;
        auto row_of = [&](int y) {
            if (!INNER && yw) {
                if (y < 0) y += ny;
                if (y >= ny) y -= ny;
                if ((unsigned)y >= (unsigned)ny) y = ((y % ny) + ny) % ny;
            }
            return y;
        };
        auto lid_row = [&](int y) { return !INNER && cavity && y == ny - 1; };
        auto pull_row = [&](int y, T (&r)[9]) {
            const int gy = row_of(y);
            if (lid_row(gy)) return;  // the lid row loads nothing
            int ym = gy - 1, yp = gy + 1;
            if (!INNER) {
                const Nb n = neighbours(0, gy, 1, ny, bc);  // rows only
                ym = n.ym;
                yp = n.yp;
            }
            pull9_row_u<ST, 0>(src, P, gy, ym, yp, pitch, cols.cc, cols.cm, cols.cp, r);
        };
        // First and last row stage s computes: the tile's and K - s beyond it.
        auto first_row = [&](int s) { return INNER || yw ? y0 - (K - s) : max(0, y0 - (K - s)); };
        auto last_row = [&](int s) { return INNER || yw ? yn - 1 + (K - s) : min(ny - 1, yn - 1 + (K - s)); };
        // One node of row y at step s (0-based) from its pulled populations,
        // left in storage form.
        auto node = [&](C (&f)[9], int s, int y, T (&sv)[9]) {
            int fl;
            if constexpr (INNER) fl = node9<ST, CO>(f, R_FLUID, in);
            else fl = node9_row<ST, CO>(f, xs, row_of(y), nx, ny, bc, in);
            const bool own = own_x && y >= y0 && y < yn;
            if (own && (fl & 1)) bad[s] = min(bad[s], y * nx + x);
            guarded += __popcll(__ballot(own && (fl & 2)));
#pragma unroll
            for (int q = 0; q < 9; ++q) sv[q] = to_storage<ST>(f[q], ref[q], a.fp16_scale);
        };
        auto lid = [&](T (&sv)[9]) {
            asm volatile("");  // a block of its own
            const double *v = lat.lid;
            // a table's values are read here, not kept in registers for every row
            if constexpr (BATCH) asm volatile("" : "+s"(v));
#pragma unroll
            for (int q = 0; q < 9; ++q) sv[q] = to_storage_apart<ST>(C(v[q]), ref[q], a.fp16_scale);
        };

        T raw[9];
        pull_row(first_row(1), raw);
        StageRows<T> st[K - 1] = {};
        for (int r = first_row(1); r < yn + K - 1; ++r) {
            T sv[9];  // the row the last stage computed
            if (r <= last_row(1)) {
                if (lid_row(r)) {
                    lid(sv);
                } else {
                    C f[9];
#pragma unroll
                    for (int q = 0; q < 9; ++q) f[q] = load<ST>(&raw[q], ref[q], a.fp16_iscale);
                    node(f, 0, r, sv);
                }
                if (r + 1 <= last_row(1)) pull_row(r + 1, raw);  // completes during the other stages
                if (BATCH && kdo == 1 && own_x && r >= y0 && r < yn) push9_xy_st<ST>(dst, P, x, r, pitch, sv);
            }
#pragma unroll
            for (int s = 1; s < K; ++s) {
                // Stage s + 1: row y from stage s, whose row y + 1 is in sv
                // (unless y is the top row).
                StageRows<T> &d = st[s - 1];
                const int y = r - s;
                if (BATCH && s >= kdo) break;
                const bool run = y >= first_row(s + 1) && y <= last_row(s + 1);
                T n4 = sv[4], n7 = lane_shift<false>(sv[7]), n8 = lane_shift<true>(sv[8]);
                T t1 = lane_shift<true>(sv[1]), t3 = lane_shift<false>(sv[3]);
                T t5 = lane_shift<true>(sv[5]), t6 = lane_shift<false>(sv[6]);
                const T t0 = sv[0], t2 = sv[2];
                if constexpr (!INNER) {
                    if (edge) {  // end nodes pull from themselves
                        n7 = at_right ? sv[7] : n7;
                        t3 = at_right ? sv[3] : t3;
                        t6 = at_right ? sv[6] : t6;
                        n8 = at_left ? sv[8] : n8;
                        t1 = at_left ? sv[1] : t1;
                        t5 = at_left ? sv[5] : t5;
                    }
                    if (y + 1 > last_row(s)) {  // beyond a top wall: the wall row's own values
                        n4 = d.a4;
                        n7 = d.a7;
                        n8 = d.a8;
                    }
                }
                if (run) {
                    if (lid_row(y)) {
                        lid(sv);
                    } else {
                        const bool bottom = !INNER && !yw && y == 0;  // the wall row pulls from itself
                        const T p2 = bottom ? d.a2 : d.b2, p5 = bottom ? d.a5 : d.b5, p6 = bottom ? d.a6 : d.b6;
                        C f[9];
                        f[0] = load<ST>(&d.a0, ref[0], a.fp16_iscale);
                        f[1] = load<ST>(&d.a1, ref[1], a.fp16_iscale);
                        f[2] = load<ST>(&p2, ref[2], a.fp16_iscale);
                        f[3] = load<ST>(&d.a3, ref[3], a.fp16_iscale);
                        f[4] = load<ST>(&n4, ref[4], a.fp16_iscale);
                        f[5] = load<ST>(&p5, ref[5], a.fp16_iscale);
                        f[6] = load<ST>(&p6, ref[6], a.fp16_iscale);
                        f[7] = load<ST>(&n7, ref[7], a.fp16_iscale);
                        f[8] = load<ST>(&n8, ref[8], a.fp16_iscale);
                        node(f, s, y, sv);
                    }
                    if (BATCH) {
                        if (s == kdo - 1 && own_x && y >= y0 && y < yn) push9_xy_st<ST>(dst, P, x, y, pitch, sv);
                    } else if (s == K - 1) {
                        if (own_x) push9_xy_st<ST>(dst, P, x, y, pitch, sv);
                    }
                }
                d.b2 = d.a2;
                d.b5 = d.a5;
                d.b6 = d.a6;
                d.a0 = t0;
                d.a1 = t1;
                d.a2 = t2;
                d.a3 = t3;
                d.a5 = t5;
                d.a6 = t6;
                if constexpr (!INNER) {
                    d.a4 = n4;
                    d.a7 = n7;
                    d.a8 = n8;
                }
            }
        }
    };
    if (!edge && y0 - K >= 0 && yn - 1 + K <= ny - 1) walk(std::true_type{});
    else walk(std::false_type{});
#pragma unroll
    for (int s = 0; s < K; ++s) report(a.status + ii, bad[s], s == 0 ? guarded : 0, a.step + s, a.step_base);
}

}  // namespace lbm
