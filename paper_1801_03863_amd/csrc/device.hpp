// device.hpp -- device code shared by the kernels of MinxEnt-LBM for gfx950:
// storage forms, pulls and stores of a node's populations, node roles, the
// status records, tile orders and the LDS barriers.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "collide.hpp"
#include "kernels.hpp"

namespace lbm {


// --------------------------------------------------------------------------
// Storage forms
// --------------------------------------------------------------------------

template <int ST> struct Form;
template <> struct Form<ST_F64> { using T = double; using C = double; };
template <> struct Form<ST_F32N64> { using T = float; using C = double; };
template <> struct Form<ST_F32> { using T = float; using C = float; };
template <> struct Form<ST_F16DEV> { using T = _Float16; using C = float; };

template <int ST>
__device__ __forceinline__ typename Form<ST>::C load(const typename Form<ST>::T *p, typename Form<ST>::C ref,
                                                     float iscale)
{
    using C = typename Form<ST>::C;
    if constexpr (ST == ST_F16DEV) return ref + C(*p) * iscale;
    else return C(*p);
}

// Raw load of one stored population; NT marks it non-temporal (streamed:
// every population is read once per step).
template <class T, bool NT>
__device__ __forceinline__ T ldraw(const T *p)
{
    if constexpr (NT) return __builtin_nontemporal_load(p);
    else return *p;
}

// Sixteen bytes of stored populations, moved as one vector access.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// The same sixteen bytes viewed as elements.
template <class T>
struct Chunk {
    T e[16 / sizeof(T)];
};

// FP16 deviation of v from ref, scaled by the power of two `scale`: the
// fused form v*scale - ref*scale rounds once, straight to binary16 (one
// mixed-precision fma); ref*scale is exact and uniform across the wave.
__device__ __forceinline__ _Float16 enc16(float v, float ref, float scale)
{
    return (_Float16)__builtin_fmaf(v, scale, -(ref * scale));
}

// A population in its storage form (rounded to the storage type, or the
// scaled FP16 deviation).
template <int ST>
__device__ __forceinline__ typename Form<ST>::T to_storage(typename Form<ST>::C v, typename Form<ST>::C ref,
                                                           float scale)
{
    using T = typename Form<ST>::T;
    if constexpr (ST == ST_F16DEV) return enc16(v, ref, scale);
    else return T(v);
}

// The same on a path beside another that converts too (the lid's rows).  Where
// such paths meet, the compiler otherwise takes the conversion out of both, and an
// FP16 deviation is rounded to float first: a kernel with such a path then differs
// from one without in the last bit of populations far from ref.  The empty
// statement keeps the conversion here, beside its fma, and so the other path's.
template <int ST>
__device__ __forceinline__ typename Form<ST>::T to_storage_apart(typename Form<ST>::C v, typename Form<ST>::C ref,
                                                                 float scale)
{
    typename Form<ST>::T t = to_storage<ST>(v, ref, scale);
    if constexpr (ST == ST_F16DEV) asm("" : "+v"(t));
    return t;
}

template <int ST, bool NT = false>
__device__ __forceinline__ void store(typename Form<ST>::T *p, typename Form<ST>::C v, typename Form<ST>::C ref,
                                      float scale)
{
    const typename Form<ST>::T t = to_storage<ST>(v, ref, scale);
    if constexpr (NT) __builtin_nontemporal_store(t, p);
    else *p = t;
}

template <class C>
__device__ __forceinline__ void ref9(C rho0, C (&r)[9])
{
    r[0] = W9<C>::rest * rho0;
#pragma unroll
    for (int a = 1; a < 5; ++a) r[a] = W9<C>::axis * rho0;
#pragma unroll
    for (int a = 5; a < 9; ++a) r[a] = W9<C>::diag * rho0;
}

// D2Q9 direction table (pull offsets are the negated velocities).
__device__ __forceinline__ int cx9(int a) { return (a == 1 || a == 5 || a == 8) ? 1 : (a == 3 || a == 6 || a == 7) ? -1 : 0; }
__device__ __forceinline__ int cy9(int a) { return (a == 2 || a == 5 || a == 6) ? 1 : (a == 4 || a == 7 || a == 8) ? -1 : 0; }

// Neighbour rows and columns of (x, y): wrapped on periodic axes, clamped
// otherwise.
struct Nb {
    int xm, xp, ym, yp;
};

__device__ __forceinline__ Nb neighbours(int x, int y, int nx, int ny, int bc)
{
    const bool xw = bc == BC_PERIODIC;
    const bool yw = bc == BC_PERIODIC || bc == BC_TUBE;
    Nb n;
    n.xm = x > 0 ? x - 1 : (xw ? nx - 1 : 0);
    n.xp = x < nx - 1 ? x + 1 : (xw ? 0 : nx - 1);
    n.ym = y > 0 ? y - 1 : (yw ? ny - 1 : 0);
    n.yp = y < ny - 1 ? y + 1 : (yw ? 0 : ny - 1);
    return n;
}

enum Role { R_FLUID = 0, R_WALL = 1, R_LID = 2 };

__device__ __forceinline__ int role9(int x, int y, int nx, int ny, int bc)
{
    switch (bc) {
    case BC_CAVITY:
        if (y == ny - 1) return R_LID;
        return (x == 0 || x == nx - 1 || y == 0) ? R_WALL : R_FLUID;
    case BC_BOX:
        return (x == 0 || x == nx - 1 || y == 0 || y == ny - 1) ? R_WALL : R_FLUID;
    case BC_TUBE:
        return (x == 0 || x == nx - 1) ? R_WALL : R_FLUID;
    default:
        return R_FLUID;
    }
}

// Pull the nine raw populations of node (x, y) given the column byte offsets
// of x and of its two neighbours.  Row bases are uniform when the rows are
// (scalar registers), so the loads take the scalar-base + 32-bit
// vector-offset form.
// NL selects non-temporal loads: 0 none, 1 every plane, 2 only the three
// planes without a horizontal shift (rest, N, S), whose cache lines no other
// tile reads; the six x-shifted planes then keep regular loads, so the line a
// tile shares with its horizontal neighbour can still be found in cache.
template <int ST, int NL = 0>
__device__ __forceinline__ void pull9_cols(const typename Form<ST>::T *__restrict__ s, int64_t P, int y, int ym,
                                           int yp, int pitch, uint32_t cc, uint32_t cm, uint32_t cp,
                                           typename Form<ST>::T (&r)[9])
{
    using T = typename Form<ST>::T;
    constexpr bool A = NL == 1, U = NL != 0;
    const int64_t PB = P * (int64_t)sizeof(T);
    const int64_t RB = (int64_t)pitch * (int64_t)sizeof(T);
    const char *bc_ = (const char *)s + (int64_t)y * RB;
    const char *bm_ = (const char *)s + (int64_t)ym * RB;
    const char *bp_ = (const char *)s + (int64_t)yp * RB;
    r[0] = ldraw<T, U>((const T *)(bc_ + cc));
    r[1] = ldraw<T, A>((const T *)((bc_ + PB) + cm));
    r[2] = ldraw<T, U>((const T *)((bm_ + 2 * PB) + cc));
    r[3] = ldraw<T, A>((const T *)((bc_ + 3 * PB) + cp));
    r[4] = ldraw<T, U>((const T *)((bp_ + 4 * PB) + cc));
    r[5] = ldraw<T, A>((const T *)((bm_ + 5 * PB) + cm));
    r[6] = ldraw<T, A>((const T *)((bm_ + 6 * PB) + cp));
    r[7] = ldraw<T, A>((const T *)((bp_ + 7 * PB) + cp));
    r[8] = ldraw<T, A>((const T *)((bp_ + 8 * PB) + cm));
}

// Non-temporal load mode of a launch-shape bit mask NT: bit 0 every plane,
// bit 2 the unshifted planes only (bit 1 is the stores; bit 3, in the
// single-lattice D2Q9 kernel, raises the wave's issue priority while it
// issues its loads).
constexpr int nl_mode(int nt) { return (nt & 1) ? 1 : ((nt & 4) ? 2 : 0); }

// Column byte offsets of a node's own column and its two neighbours.  In a
// tile that touches neither side of the lattice the neighbours are x -+ 1
// for every boundary kind, so only the two edge tiles of a row (a uniform
// test) evaluate the wrap/clamp rule.
struct Cols {
    uint32_t cc, cm, cp;
};

__device__ __forceinline__ Cols columns(int xs, bool edge_tile, int nx, int bc, uint32_t E)
{
    Cols c;
    c.cc = (uint32_t)xs * E;
    c.cm = c.cc - E;
    c.cp = c.cc + E;
    if (edge_tile) {
        const Nb n = neighbours(xs, 0, nx, 1, bc);
        c.cm = (uint32_t)n.xm * E;
        c.cp = (uint32_t)n.xp * E;
    }
    return c;
}

// Pull the nine raw stored populations that stream into node (x, y) (rows
// `pitch` elements apart).
template <int ST, int NL = 0>
__device__ __forceinline__ void pull9_raw(const typename Form<ST>::T *__restrict__ s, int64_t P, int x, int y,
                                          int pitch, const Nb &n, typename Form<ST>::T (&r)[9])
{
    const uint32_t E = sizeof(typename Form<ST>::T);
    pull9_cols<ST, NL>(s, P, y, n.ym, n.yp, pitch, (uint32_t)x * E, (uint32_t)n.xm * E, (uint32_t)n.xp * E, r);
}

// Pull and widen the nine populations that stream into node (x, y) (NL as
// for pull9_cols).
template <int ST, int NL = 0>
__device__ __forceinline__ void pull9(const typename Form<ST>::T *__restrict__ s, int64_t P, int x, int y,
                                      int pitch, const Nb &n, const typename Form<ST>::C (&ref)[9], float iscale,
                                      typename Form<ST>::C (&f)[9])
{
    typename Form<ST>::T r[9];
    pull9_raw<ST, NL>(s, P, x, y, pitch, n, r);
#pragma unroll
    for (int q = 0; q < 9; ++q) f[q] = load<ST>(&r[q], ref[q], iscale);
}

// Write the nine populations of node (x, y), already in their storage form,
// of a row that is uniform across the wave.  The row base is read from the
// first lane so that it lives in scalar registers, and each store takes the
// scalar-base + 32-bit vector-offset form of a global store.
template <int ST, bool NT = false>
__device__ __forceinline__ void push9_xy_st(typename Form<ST>::T *__restrict__ d, int64_t P, int x, int y,
                                            int pitch, const typename Form<ST>::T (&v)[9])
{
    using T = typename Form<ST>::T;
    using GT = __attribute__((address_space(1))) T;
    const uint64_t a = (uint64_t)d + (uint64_t)((int64_t)y * pitch * (int64_t)sizeof(T));
    // readfirstlane returns a signed int: each half goes through uint32_t so
    // that widening zero-extends it.
    const uint32_t ahi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(a >> 32));
    const uint32_t alo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    const uint64_t b = ((uint64_t)ahi << 32) | (uint64_t)alo;
    const uint64_t PB = (uint64_t)P * sizeof(T);
    // The empty asm statements keep the lane offset and each plane base
    // opaque, so the compiler can neither share a widened offset with the
    // loads nor fold it into a 64-bit vector address.
    uint32_t o = (uint32_t)x * (uint32_t)sizeof(T);
    asm volatile("" : "+v"(o));
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        uint64_t bq = b + q * PB;
        asm volatile("" : "+s"(bq));
        GT *p = (GT *)(bq + (uint64_t)o);
        if constexpr (NT) __builtin_nontemporal_store(v[q], p);
        else *p = v[q];
    }
}

// The same from populations in compute precision.
template <int ST, bool NT = false>
__device__ __forceinline__ void push9_xy(typename Form<ST>::T *__restrict__ d, int64_t P, int x, int y,
                                         int pitch, const typename Form<ST>::C (&f)[9],
                                         const typename Form<ST>::C (&ref)[9], float scale)
{
    typename Form<ST>::T v[9];
#pragma unroll
    for (int q = 0; q < 9; ++q) v[q] = to_storage<ST>(f[q], ref[q], scale);
    push9_xy_st<ST, NT>(d, P, x, y, pitch, v);
}

// Address of a block-uniform pointer, read from the first lane so that it
// lives in scalar registers (each half through uint32_t: readfirstlane
// returns a signed int, and widening must zero-extend it).
__device__ __forceinline__ uint64_t uniform_addr(const void *p)
{
    const uint64_t v = (uint64_t)p;
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(v >> 32));
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)v);
    return ((uint64_t)hi << 32) | (uint64_t)lo;
}

// Batched D2Q9: pull the nine raw populations of a node of one instance,
// whose planes start at the block-uniform address s (stride P elements),
// from byte offsets of rows (rc own, rm below, rp above) and columns (cc
// own, cm left, cp right).  An instance holds fewer than 2^22 nodes and
// pads each row by fewer than 64 elements, so its plane spans fewer than
// 2^28 elements (2^31 bytes) and every offset fits 32 bits: each load takes
// the scalar-base + 32-bit vector-offset form.  NL as for pull9_cols.
template <int ST, int NL>
__device__ __forceinline__ void pull9_inst(uint64_t s, int64_t P, uint32_t rc, uint32_t rm, uint32_t rp,
                                           uint32_t cc, uint32_t cm, uint32_t cp, typename Form<ST>::T (&r)[9])
{
    using T = typename Form<ST>::T;
    using GT = const __attribute__((address_space(1))) T;
    constexpr bool A = NL == 1, U = NL != 0;
    constexpr bool nt[9] = {U, A, U, A, U, A, A, A, A};
    const uint32_t o[9] = {rc + cc, rc + cm, rm + cc, rc + cp, rp + cc, rm + cm, rm + cp, rp + cp, rp + cm};
    const uint64_t PB = (uint64_t)P * sizeof(T);
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        uint64_t bq = s + q * PB;
        asm volatile("" : "+s"(bq));
        uint32_t oq = o[q];
        asm volatile("" : "+v"(oq));
        GT *p = (GT *)(bq + (uint64_t)oq);
        if (nt[q]) r[q] = __builtin_nontemporal_load(p);
        else r[q] = *p;
    }
}

// Pull of a row that is uniform across the block (the two-step kernel's
// window rows): rows y (own), ym (below), yp (above), columns as byte
// offsets cc, cm, cp.  Each row and plane base lives in scalar registers and
// each load takes the scalar-base + 32-bit vector-offset form, so no lane
// forms a 64-bit address.  NL as for pull9_cols.
template <int ST, int NL>
__device__ __forceinline__ void pull9_row_u(const typename Form<ST>::T *__restrict__ s, int64_t P, int y, int ym,
                                            int yp, int pitch, uint32_t cc, uint32_t cm, uint32_t cp,
                                            typename Form<ST>::T (&r)[9])
{
    using T = typename Form<ST>::T;
    using GT = const __attribute__((address_space(1))) T;
    constexpr bool A = NL == 1, U = NL != 0;
    constexpr bool nt[9] = {U, A, U, A, U, A, A, A, A};
    constexpr int row[9] = {0, 0, 1, 0, 2, 1, 1, 2, 2};  // own, below, above
    constexpr int col[9] = {0, 1, 0, 2, 0, 1, 2, 2, 1};  // own, left, right
    const uint64_t s0 = uniform_addr(s);
    const uint64_t RB = (uint64_t)pitch * sizeof(T), PB = (uint64_t)P * sizeof(T);
    const uint64_t rb[3] = {s0 + (uint64_t)y * RB, s0 + (uint64_t)ym * RB, s0 + (uint64_t)yp * RB};
    uint32_t co[3] = {cc, cm, cp};
    asm volatile("" : "+v"(co[0]), "+v"(co[1]), "+v"(co[2]));
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        uint64_t bq = rb[row[q]] + q * PB;
        asm volatile("" : "+s"(bq));
        GT *p = (GT *)(bq + (uint64_t)co[col[q]]);
        if (nt[q]) r[q] = __builtin_nontemporal_load(p);
        else r[q] = *p;
    }
}

// Batched D2Q9: write the nine populations of the node at byte offset o of
// the instance whose planes start at the block-uniform address d.
template <int ST, bool NT = false>
__device__ __forceinline__ void push9_inst(uint64_t d, int64_t P, uint32_t o, const typename Form<ST>::C (&f)[9],
                                           const typename Form<ST>::C (&ref)[9], float scale)
{
    using T = typename Form<ST>::T;
    using GT = __attribute__((address_space(1))) T;
    const uint64_t PB = (uint64_t)P * sizeof(T);
    asm volatile("" : "+v"(o));
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        uint64_t bq = d + q * PB;
        asm volatile("" : "+s"(bq));
        GT *p = (GT *)(bq + (uint64_t)o);
        T t;
        if constexpr (ST == ST_F16DEV) t = enc16(f[q], ref[q], scale);
        else t = T(f[q]);
        if constexpr (NT) __builtin_nontemporal_store(t, p);
        else *p = t;
    }
}

// Role collision of one D2Q9 node.  Returns bit 0 = unstable, bit 1 = guarded.
template <int ST, int CO>
__device__ __forceinline__ int node9(typename Form<ST>::C (&f)[9], int role, const Inst &in)
{
    using C = typename Form<ST>::C;
    if (role == R_LID) {
#pragma unroll
        for (int a = 0; a < 9; ++a) f[a] = C(in.lid[a]);
        return 0;
    }
    if constexpr (ST == ST_F16DEV && (CO == CO_MINXENT4 || CO == CO_MINXENT2)) {
        // FP16 deviations: the collision runs on the fluid lanes only, then
        // the wall lanes, whose f still holds the pulled populations, swap
        // them.  The same results as the order below; in this form the
        // compiler then keeps fewer values live across the collision (69
        // instead of 77 VGPRs in the tuned two-step shape, 7 waves per SIMD
        // instead of 6).  In the double-precision forms this order costs
        // registers instead.
        int r = 0;
        if (role != R_WALL) {
            bool ok = true;
            const bool g = collide_minxent<C, CO == CO_MINXENT2, true, false>(f, C(in.omega), C(in.omega2), ok);
            r = (g ? 2 : 0) | (ok ? 0 : 1);
        }
        if (role == R_WALL) {
            C t;
            t = f[1]; f[1] = f[3]; f[3] = t;
            t = f[2]; f[2] = f[4]; f[4] = t;
            t = f[5]; f[5] = f[7]; f[7] = t;
            t = f[6]; f[6] = f[8]; f[8] = t;
        }
        return r;
    }
    if (role == R_WALL) {
        C t;
        t = f[1]; f[1] = f[3]; f[3] = t;
        t = f[2]; f[2] = f[4]; f[4] = t;
        t = f[5]; f[5] = f[7]; f[7] = t;
        t = f[6]; f[6] = f[8]; f[8] = t;
        return 0;
    }
    // Stable iff every population is >= 0 and finite (Sec. IV.G): the
    // minimum catches negatives; inf and NaN are caught by the Newton
    // increments (MinxEnt) or by the sum (the other rules).
    if constexpr (CO == CO_MINXENT4 || CO == CO_MINXENT2) {
        bool ok = true;
        const bool g = collide_minxent<C, CO == CO_MINXENT2, ST == ST_F16DEV, ST == ST_F32N64>(f, C(in.omega), C(in.omega2), ok);
        return (g ? 2 : 0) | (ok ? 0 : 1);
    } else {
        if constexpr (CO == CO_SRT) {
            collide_srt<C>(f, C(in.omega));
        } else if constexpr (CO == CO_TRT) {
            collide_mrt<C>(f, C(in.omega), C(in.omega), C(in.omega2), C(in.omega));
        } else {
            collide_mrt<C>(f, C(1.64), C(1.54), C(in.omega2), C(in.omega));
        }
        C mn = f[0], sm = f[0];
#pragma unroll
        for (int a = 1; a < 9; ++a) {
            mn = __builtin_fmin(mn, f[a]);
            sm += f[a];
        }
        const bool ok = mn >= C(0) && sm < C(__builtin_huge_valf());
        return ok ? 0 : 1;
    }
}

// Role collision of one node of a non-lid row that is uniform across the
// wave: only the two side-wall lanes diverge.
template <int ST, int CO>
__device__ __forceinline__ int node9_row(typename Form<ST>::C (&f)[9], int x, int y, int nx, int ny, int bc,
                                         const Inst &in)
{
    const bool wall_row = (bc == BC_CAVITY && y == 0) || (bc == BC_BOX && (y == 0 || y == ny - 1));
    const bool wall = wall_row || (bc != BC_PERIODIC && (x == 0 || x == nx - 1));
    return node9<ST, CO>(f, wall ? R_WALL : R_FLUID, in);
}

// The cavity's lid row (uniform across the wave): every node takes the lid
// equilibrium, which needs no loads.
template <int ST, bool NT = false>
__device__ __forceinline__ void push_lid(typename Form<ST>::T *__restrict__ d, int64_t P, int x, int y, int pitch,
                                         const Inst &in, const typename Form<ST>::C (&ref)[9], float scale)
{
    using C = typename Form<ST>::C;
    typename Form<ST>::T v[9];
#pragma unroll
    for (int a = 0; a < 9; ++a) v[a] = to_storage_apart<ST>(C(in.lid[a]), ref[a], scale);
    push9_xy_st<ST, NT>(d, P, x, y, pitch, v);
}

// Key of an unstable event: the step in the high word (saturating at 2^32 -
// 1), the node index (x + y nx within its instance) in the low word, so that
// the smallest key is the first step's smallest node.
__device__ __forceinline__ uint64_t event_key(int64_t step, int node)
{
    const uint64_t s = step < 0xffffffffll ? (uint64_t)step : 0xffffffffull;
    return (s << 32) | (uint32_t)node;
}

// Sentinel of a lane's unstable-node record: no unstable node.
constexpr int kNoNode = 0x7fffffff;

// bad_node: the smallest unstable node index of this lane in this launch, or
// kNoNode.  One atomic per wave and kind; the wave's smallest unstable node
// is found by a butterfly minimum only in waves that have one.
__device__ __forceinline__ void report(DevStatus *st, int bad_node, int guarded_in_wave, int64_t step,
                                       const int64_t *step_base)
{
    const unsigned long long m = __ballot(bad_node != kNoNode);
    if (m != 0ull) {
        int v = bad_node;
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) v = min(v, __shfl_xor(v, o));
        if (__lane_id() == 0) {
            const int64_t s = step + (step_base ? *step_base : 0);
            atomicOr(&st->flags, 1u);
            atomicMin((unsigned long long *)&st->first, (unsigned long long)event_key(s, v));
        }
    }
    if (guarded_in_wave != 0 && __lane_id() == 0) {
        atomicOr(&st->flags, 2u);
        atomicAdd((unsigned long long *)&st->guarded, (unsigned long long)guarded_in_wave);
    }
}

// Batched instances with a step limit: once the step index reaches the
// instance's `stop`, its launches carry the state over unchanged (the two
// buffers alternate for the whole batch).
__device__ __forceinline__ bool instance_stopped(const StepArgs &a, const Inst &in)
{
    return in.stop <= a.step + (a.step_base ? *a.step_base : 0);
}

template <class T>
__device__ __forceinline__ void carry_node(const T *__restrict__ s, T *__restrict__ d, int64_t P, int planes, int node)
{
    for (int q = 0; q < planes; ++q) d[q * P + node] = s[q * P + node];
}

// Map block b of a grid of nb blocks so that the blocks the hardware sends to
// one XCD (b, b+8, b+16, ...) cover a contiguous range of tiles.
__device__ __forceinline__ int xcd_remap(int b, int nb)
{
    const int q = nb >> 3, r = nb & 7, k = b & 7;
    return k * q + (k < r ? k : r) + (b >> 3);
}

// Tile (tx, ty) of this block.  The grid is (tiles_x, tiles_y), or one
// dimension of tiles_x * tiles_y blocks when tiles_y exceeds the grid's y
// limit.  In dispatch order (x fastest) the hardware deals blocks
// round-robin to the eight XCDs, each with its own L2; with the swizzle the
// linear block index is remapped so that each XCD works on a contiguous band
// of rows.
__device__ __forceinline__ void tile_of_block(int swizzle, int tiles_x, int &tx, int &ty)
{
    if (!swizzle && (int)gridDim.x == tiles_x) {
        tx = blockIdx.x;
        ty = blockIdx.y;
        return;
    }
    int b = blockIdx.y * gridDim.x + blockIdx.x;
    if (swizzle) b = xcd_remap(b, gridDim.x * gridDim.y);
    ty = b / tiles_x;
    tx = b - ty * tiles_x;
}

// Workgroup barrier that orders LDS accesses only, so global loads issued
// before it stay in flight.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The same ordering within one wave, for tiles a single wave owns: LDS
// writes before it are visible to every lane of the wave after it.
__device__ __forceinline__ void lds_wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// --------------------------------------------------------------------------
// D1Q3 (rest, +1, -1): SRT, the exact form of the method on this lattice.
// --------------------------------------------------------------------------

template <class C>
__device__ __forceinline__ void collide3(C &f0, C &fp, C &fm, C omega)
{
    const C rho = (f0 + fp) + fm;
    const C u = (fp - fm) * rcp(rho);
    const C uu = u * u;
    const C e0 = C(2.0 / 3.0) * rho * (C(1) - C(1.5) * uu);
    const C es = C(1.0 / 6.0) * rho * (C(1) + C(3) * uu);
    const C eu = C(1.0 / 6.0) * rho * (C(3) * u);
    f0 = f0 + omega * (e0 - f0);
    fp = fp + omega * ((es + eu) - fp);
    fm = fm + omega * ((es - eu) - fm);
}

template <class C>
__device__ __forceinline__ int node3(C &f0, C &fp, C &fm, int role, C omega)
{
    if (role == R_WALL) {
        const C t = fp;
        fp = fm;
        fm = t;
        return 0;
    }
    collide3(f0, fp, fm, omega);
    return (nonneg_finite(f0) && nonneg_finite(fp) && nonneg_finite(fm)) ? 0 : 1;
}

// The value of the lane below (left neighbour column) or above; lanes 0 and
// 63 keep their own, which only dead columns use.
template <bool FROM_LEFT>
__device__ __forceinline__ uint32_t wave_shift(uint32_t v)
{
    constexpr int ctrl = FROM_LEFT ? 0x138 : 0x130;  // wave_shr:1, wave_shl:1
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, ctrl, 0xf, 0xf, false);
}
template <bool FROM_LEFT>
__device__ __forceinline__ float lane_shift(float v)
{
    return __builtin_bit_cast(float, wave_shift<FROM_LEFT>(__builtin_bit_cast(uint32_t, v)));
}
template <bool FROM_LEFT>
__device__ __forceinline__ double lane_shift(double v)
{
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const uint32_t lo = wave_shift<FROM_LEFT>((uint32_t)u), hi = wave_shift<FROM_LEFT>((uint32_t)(u >> 32));
    return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
template <bool FROM_LEFT>
__device__ __forceinline__ _Float16 lane_shift(_Float16 v)
{
    return __builtin_bit_cast(_Float16,
                              (uint16_t)wave_shift<FROM_LEFT>((uint32_t)__builtin_bit_cast(uint16_t, v)));
}

// Wave-level minimum of a 64-bit event key and one atomic for the wave.
__device__ __forceinline__ void report_key(DevStatus *st, uint64_t key)
{
    if (__ballot(key != ~0ull) == 0ull) return;
    uint32_t lo = (uint32_t)key, hi = (uint32_t)(key >> 32);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const uint32_t l2 = (uint32_t)__shfl_xor((int)lo, o), h2 = (uint32_t)__shfl_xor((int)hi, o);
        if (h2 < hi || (h2 == hi && l2 < lo)) {
            hi = h2;
            lo = l2;
        }
    }
    if (__lane_id() == 0) {
        atomicOr(&st->flags, 1u);
        atomicMin((unsigned long long *)&st->first, ((unsigned long long)hi << 32) | lo);
    }
}

}  // namespace lbm
