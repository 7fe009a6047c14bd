// ot_interact.h -- device side of the interaction kernels: sub-grid geometry,
// the compile-time stencil table, per-pair arithmetic, LDS staging and the
// k_interact kernel template. Included once, by ot_fmm.hip (host side and
// C ABI). The design notes are at the top of ot_fmm.hip.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <atomic>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <numeric>
#include <string>
#include <utility>
#include <vector>

#include "ot_common.h"
#include "ot_fmm.h"
#include "ot_pair.h"

using namespace otfmm;

namespace {

// ---------------------------------------------------------------------------
// Stencil: for target parity (0, 0, pz), the offsets d = j - i grouped into
// rows (dz, dy, [dx0, dx0 + n)). Built at compile time from the criterion.
// Targets of x (y) parity 1 use the same rows with dx (dy) negated.
// ---------------------------------------------------------------------------
constexpr int floor_half(int v) { return v >= 0 ? v / 2 : -((-v + 1) / 2); }

constexpr bool criterion(int ix, int iy, int iz, int jx, int jy, int jz)
{
    const int dx = jx - ix, dy = jy - iy, dz = jz - iz;
    const int px = floor_half(jx) - floor_half(ix), py = floor_half(jy) - floor_half(iy),
              pz = floor_half(jz) - floor_half(iz);
    return dx * dx + dy * dy + dz * dz > 16 && px * px + py * py + pz * pz <= 16;
}

struct StencilTable {
    uint32_t rows[2][kMaxRows];           // packed: dy | dx0 << 8 | n << 16
    int range[2][2 * kReach + 1][2];      // per (pz, dz+9): first row, end row
    int count[2];                         // offsets per parity (1799)
};

constexpr uint32_t pack_row(int dy, int dx0, int n)
{
    return (uint32_t)(dy & 0xff) | ((uint32_t)(dx0 & 0xff) << 8) | ((uint32_t)n << 16);
}

constexpr StencilTable build_stencil()
{
    StencilTable t{};
    for (int pz = 0; pz < 2; ++pz) {
        const int ix = 8, iy = 8, iz = 8 + pz;
        int nr = 0, total = 0;
        for (int dz = -kReach; dz <= kReach; ++dz) {
            const int first = nr;
            int offs = 0;
            for (int dy = -kReach; dy <= kReach; ++dy) {
                int dx = -kReach;
                while (dx <= kReach) {
                    if (!criterion(ix, iy, iz, ix + dx, iy + dy, iz + dz)) {
                        ++dx;
                        continue;
                    }
                    int n = 0;
                    while (dx + n <= kReach && criterion(ix, iy, iz, ix + dx + n, iy + dy, iz + dz))
                        ++n;
                    t.rows[pz][nr++] = pack_row(dy, dx, n);
                    offs += n;
                    dx += n;
                }
            }
            t.range[pz][dz + kReach][0] = first;
            t.range[pz][dz + kReach][1] = nr;
            total += offs;
        }
        t.count[pz] = total;
    }
    return t;
}

constexpr StencilTable kStencilHost = build_stencil();
static_assert(kStencilHost.count[0] == 1799 && kStencilHost.count[1] == 1799, "stencil size");

// Exact number of pairs between the 8^3 target cells and the neighbour block
// at each slot, plus a check that the mirrored table reproduces the stencil
// of every parity. Computed once on the host.
struct SlotCounts {
    int64_t pairs[27];
    bool mirror_ok;
};

SlotCounts compute_slot_counts()
{
    SlotCounts sc{};
    for (int slot = 0; slot < 27; ++slot) {
        const int ox = 8 * (slot % 3), oy = 8 * ((slot / 3) % 3), oz = 8 * (slot / 9);
        int64_t n = 0;
        for (int i = 0; i < kSub3; ++i) {
            const int ix = 8 + i % 8, iy = 8 + (i / 8) % 8, iz = 8 + i / 64;
            for (int j = 0; j < kSub3; ++j)
                n += criterion(ix, iy, iz, ox + j % 8, oy + (j / 8) % 8, oz + j / 64);
        }
        sc.pairs[slot] = n;
    }
    // every parity's brute-force stencil == mirrored rows of its z-parity
    bool ok = true;
    for (int p = 0; p < 8 && ok; ++p) {
        const int px = p & 1, py = (p >> 1) & 1, pz = p >> 2;
        const int ix = 8 + px, iy = 8 + py, iz = 8 + pz;
        static bool mark[19][19][19];
        std::memset(mark, 0, sizeof(mark));
        int n_table = 0;
        for (int dz = -kReach; dz <= kReach; ++dz) {
            const int* rg = kStencilHost.range[pz][dz + kReach];
            for (int r = rg[0]; r < rg[1]; ++r) {
                const uint32_t w = kStencilHost.rows[pz][r];
                const int dy = (int8_t)(w & 0xff), dx0 = (int8_t)((w >> 8) & 0xff), n = (int)(w >> 16);
                for (int k = 0; k < n; ++k) {
                    const int dx = (px ? -1 : 1) * (dx0 + k), dyy = (py ? -1 : 1) * dy;
                    if (!criterion(ix, iy, iz, ix + dx, iy + dyy, iz + dz)) ok = false;
                    mark[dz + 9][dyy + 9][dx + 9] = true;
                    ++n_table;
                }
            }
        }
        int n_brute = 0;
        for (int dz = -kReach; dz <= kReach; ++dz)
            for (int dy = -kReach; dy <= kReach; ++dy)
                for (int dx = -kReach; dx <= kReach; ++dx)
                    if (criterion(ix, iy, iz, ix + dx, iy + dy, iz + dz)) {
                        ++n_brute;
                        if (!mark[dz + 9][dy + 9][dx + 9]) ok = false;
                    }
        if (n_brute != n_table) ok = false;
    }
    sc.mirror_ok = ok;
    return sc;
}

const SlotCounts& slot_counts()
{
    static const SlotCounts sc = compute_slot_counts();
    return sc;
}

// ---------------------------------------------------------------------------
// Kept outputs: within a group of outputs of one order and one truncation,
// every output whose z exponent is 2 or more follows from two others,
// L_{g+zz} = -(L_{g+xx} + L_{g+yy}) (the derivatives of 1/r are trace-free),
// and is rebuilt after the sum.
// ---------------------------------------------------------------------------
__host__ __device__ constexpr bool kept(int g) { return exp_of(g).c < 2; }

// position of a kept multi-index among the kept ones of [lo, g)
__host__ __device__ constexpr int kept_slot(int lo, int g)
{
    int n = 0;
    for (int h = lo; h < g; ++h) n += kept(h) ? 1 : 0;
    return n;
}

static_assert(kept_slot(0, 20) == 16 && kept_slot(1, 35) == 24, "kept outputs");

// full[g - LO] for g in [LO, LO + sizeof...(I)) from the kept accumulators;
// outputs with z exponent >= 2 are rebuilt in index order (their two
// partners always come earlier in graded-lex order).
template <int LO, int G_>
__device__ __forceinline__ void expand_one(const double* acc, double* full)
{
    if constexpr (kept(G_)) {
        constexpr int slot = kept_slot(LO, G_);
        full[G_ - LO] = acc[slot];
    } else {
        constexpr Exp3 e = exp_of(G_);
        constexpr int gx = idx_of(e.a + 2, e.b, e.c - 2);
        constexpr int gy = idx_of(e.a, e.b + 2, e.c - 2);
        full[G_ - LO] = -(full[gx - LO] + full[gy - LO]);
    }
}
template <int LO, int... I>
__device__ __forceinline__ void expand(const double* acc, double* full, std::integer_sequence<int, I...>)
{
    (expand_one<LO, LO + I>(acc, full), ...);
}

// Adjoint epilogue: with C_g (g = 1..34, stored at C[g - 1]) the derivative
// sums of orders 1..4 -- L'_g for the target role, F_g + E_g (E_g alone for
// |g| = 4) for the source role -- the position gradient is
// gX_k = sum_a c_a C_{a+e_k}, where c_a is the target's weight w_a (target
// role) or M_a / a! (source role).
template <int A, int K>
__device__ __forceinline__ double c_term(const double* C)
{
    constexpr int g = sum_idx(A, K);
    return C[g - 1];
}
template <int... A>
__device__ __forceinline__ void grad_x(const double* c, const double* C, double* gx,
                                       std::integer_sequence<int, A...>)
{
    ((gx[0] = __builtin_fma(c[A], c_term<A, 1>(C), gx[0]),
      gx[1] = __builtin_fma(c[A], c_term<A, 2>(C), gx[1]),
      gx[2] = __builtin_fma(c[A], c_term<A, 3>(C), gx[2])),
     ...);
}
// C_g = F_g + E_g for 1 <= |g| <= 3, E_g for |g| = 4 (g = I + 1)
template <int... I>
__device__ __forceinline__ void combine_fe(const double* F, const double* E, double* C,
                                           std::integer_sequence<int, I...>)
{
    ((C[I] = (I + 1 < 20) ? F[(I + 1) % 20] + E[I] : E[I]), ...);
}
template <int A>
__device__ __forceinline__ double inv_fact_c()
{
    constexpr double f = inv_multi_factorial(A);
    return f;
}
template <int... A>
__device__ __forceinline__ void scale_inv_fact(double* c, std::integer_sequence<int, A...>)
{
    ((c[A] *= inv_fact_c<A>()), ...);
}

// ---------------------------------------------------------------------------
// Kernel
// ---------------------------------------------------------------------------
enum Mode : int {
    MODE_MONO_HALO = 0,  // single block, mass only -> L
    MODE_FWD_HALO = 1,   // single block, moments -> L
    MODE_FWD_STORE = 2,  // batched forward -> L
    MODE_B2_STORE = 3,   // adjoint, source role per store sub-grid -> gM, gX (overwrite)
    MODE_B1_STORE = 4,   // adjoint, target role per target -> gX (accumulate)
    MODE_FULL_STORE = 5,  // batched forward, full truncation -> L
    MODE_B2F_STORE = 6,   // adjoint of the full truncation, source role -> gM, gX (overwrite)
    MODE_B1F_STORE = 7,   // adjoint of the full truncation, target role -> gX (accumulate)
    MODE_FS_STORE = 8,    // batched forward -> L, plus the target-role sums the adjoint needs
    MODE_B2S_STORE = 9,   // adjoint from those sums: source role per store sub-grid, plus the
                          // target role of its cells from the saved sums -> gM, gX (overwrite)
    MODE_AMC_STORE = 10,  // batched forward -> L, plus the angular-momentum correction of the
                          // force of each target cell -> dF
    MODE_FSF_STORE = 11,  // full truncation: forward -> L, plus the target-role sums of its adjoint
    MODE_B2SF_STORE = 12  // full truncation: one-pass adjoint from those sums -> gM, gX (overwrite)
};

constexpr int kMaxPieces = 16;  // work-list pieces (one per XCD) of a persistent launch

struct KParams {
    const double* mom;   // source moments / masses / weights, [ncomp][mom_stride]
    const double* pos;   // centres of mass, [3][pos_stride] (halo or store)
    long mom_stride;
    long pos_stride;
    const int4* rel;       // [owners][27]: {moment block, position block, packed shift, 0}
    const int* own_blk;    // owner -> store block of its own cells (NULL: identity)
    const int* order;      // work-group -> owner (NULL: from `first` on)
    int first;             // with no order: the first owner of the launch
    const double* aux;     // epilogue input: gL (B1) or M (B2), [20][aux_stride]
    long aux_stride;
    // B2S epilogue, the target role of the owner's cells: store sub-grid ->
    // target index (-1: none), that target's gL [20][aux_stride2] and its
    // saved sums [24][aux_stride2]
    const int* store_tgt;
    const double* aux2;
    const double* save;
    long aux_stride2;
    double* out0;          // L, or gM (B2), or gX (B1)
    double* out1;          // gX (B2), the saved target-role sums (FS) or the force correction (AMC)
    long out_stride;
    const int* out_blk;    // owner -> output block (NULL: identity)
    const int* invalid;    // forward: a count that, if not zero, makes the outputs NaN (NULL: none)
    double period[3];
    int* counter;          // persistent launch: work counter(s), zero before and after it
    int n_items;           // persistent launch: number of work-list entries
    // persistent launch in pieces (npieces > 0): the work list is cut into
    // npieces consecutive pieces, [piece_off[k], piece_off[k + 1]), one per
    // XCD, each with its own counter counter[k]
    int npieces;
    int piece_off[kMaxPieces + 1];
};

template <int MODE>
struct ModeTraits {
    static constexpr bool halo = (MODE == MODE_MONO_HALO || MODE == MODE_FWD_HALO);
    static constexpr bool adjoint = (MODE == MODE_B1_STORE || MODE == MODE_B2_STORE || MODE == MODE_B1F_STORE ||
                                     MODE == MODE_B2F_STORE || MODE == MODE_B2S_STORE || MODE == MODE_B2SF_STORE);
    static constexpr bool source_role = (MODE == MODE_B2_STORE || MODE == MODE_B2F_STORE ||
                                         MODE == MODE_B2S_STORE || MODE == MODE_B2SF_STORE);
    // one set of sums of orders 0..4 under the full truncation (every |b| <= 3)
    static constexpr bool full4 = (MODE == MODE_B2F_STORE || MODE == MODE_B2SF_STORE || MODE == MODE_FSF_STORE);
    // the target role added from saved sums in the source-role pass's epilogue
    static constexpr bool saved_target = (MODE == MODE_B2S_STORE || MODE == MODE_B2SF_STORE);
    // the F + E sums (total order 3, and the order-4 terms of orders 1..4)
    static constexpr bool fe = (MODE == MODE_B2_STORE || MODE == MODE_B2S_STORE || MODE == MODE_FS_STORE ||
                                MODE == MODE_AMC_STORE);
    // the sums a pair adds into, the staged record and the accumulators
    static constexpr int sums = (MODE == MODE_MONO_HALO)    ? SUMS_MONO
                                : (MODE == MODE_B1_STORE)   ? SUMS_T4
                                : (MODE == MODE_B1F_STORE)  ? SUMS_X4T
                                : (MODE == MODE_FULL_STORE) ? SUMS_X3
                                : fe                        ? SUMS_FE
                                : full4                     ? SUMS_X4
                                                            : SUMS_F3;
    static constexpr int nc = record_size(sums);
    static constexpr int nacc = sums_count(sums);
};

// What a target cell's finished sums become: the outputs of the mode, written
// (B1: added) at the cell's place. `acc`: the sums of cell `cell` of `owner`.
template <int MODE>
__device__ __forceinline__ void store_sums(const KParams& p, int owner, int cell, double* acc)
{
    using T = ModeTraits<MODE>;
    finish_sums<T::sums>(acc);
    if constexpr (MODE == MODE_FSF_STORE) {
        // full truncation: L is the sums of orders 0..3 (kept slots 0..15);
        // the target-role sums C'_g, 1 <= |g| <= 4, are the kept slots 1..24
        double L[20];
        expand<0>(acc, L, std::make_integer_sequence<int, 20>{});
        const long b = p.out_blk ? p.out_blk[owner] : owner;
        const long ob = b * kSub3 + cell;
#pragma unroll
        for (int a = 0; a < 20; ++a) p.out0[a * p.out_stride + ob] = L[a];
#pragma unroll
        for (int k = 0; k < 24; ++k) p.out1[k * p.out_stride + ob] = acc[k + 1];
    } else if constexpr (MODE == MODE_FS_STORE) {
        // L from F; the saved sums C'_g (1 <= |g| <= 4, total order 4) =
        // F_g + E_g for |g| <= 3, E_g for |g| = 4, in kept slots (F's kept
        // slot k + 1 and C's kept slot k are the same multi-index)
        double L[20];
        expand<0>(acc, L, std::make_integer_sequence<int, 20>{});
        const long b = p.out_blk ? p.out_blk[owner] : owner;
        const long ob = b * kSub3 + cell;
#pragma unroll
        for (int a = 0; a < 20; ++a) p.out0[a * p.out_stride + ob] = L[a];
#pragma unroll
        for (int k = 0; k < 24; ++k) p.out1[k * p.out_stride + ob] = k < 15 ? acc[k + 1] + acc[16 + k] : acc[16 + k];
    } else if constexpr (MODE == MODE_AMC_STORE) {
        // L from F; the force correction dF_k = -sum_{|a| <= 3} (M_a/a!) E_{a+e_k}
        // (E: the sums of exact total order 4), with the target cell's own moments
        double L[20];
        expand<0>(acc, L, std::make_integer_sequence<int, 20>{});
        const long b = p.out_blk ? p.out_blk[owner] : owner;
        const long ob = b * kSub3 + cell;
#pragma unroll
        for (int a = 0; a < 20; ++a) p.out0[a * p.out_stride + ob] = L[a];
        double E[34];
        expand<1>(acc + 16, E, std::make_integer_sequence<int, 34>{});
        const long mb = (p.own_blk ? p.own_blk[owner] : owner) * (long)kSub3 + cell;
        double c[20];
#pragma unroll
        for (int a = 0; a < 20; ++a) c[a] = p.aux[a * p.aux_stride + mb];
        scale_inv_fact(c, std::make_integer_sequence<int, 20>{});
        double gx[3] = {0.0, 0.0, 0.0};
        grad_x(c, E, gx, std::make_integer_sequence<int, 20>{});
#pragma unroll
        for (int k = 0; k < 3; ++k) p.out1[k * p.out_stride + ob] = -gx[k];
    } else if constexpr (!T::adjoint) {
        double L[20];
        expand<0>(acc, L, std::make_integer_sequence<int, 20>{});
        if constexpr (MODE == MODE_FWD_STORE) {
            if (p.invalid && *p.invalid != 0) {
#pragma unroll
                for (int a = 0; a < 20; ++a) L[a] = __builtin_nan("");
            }
        }
        const long b = p.out_blk ? p.out_blk[owner] : owner;
#pragma unroll
        for (int a = 0; a < 20; ++a) p.out0[a * p.out_stride + b * kSub3 + cell] = L[a];
    } else {
        double C[34];
        double F[20];
        if constexpr (MODE == MODE_B1_STORE || MODE == MODE_B1F_STORE) {
            expand<1>(acc, C, std::make_integer_sequence<int, 34>{});
        } else if constexpr (T::full4) {
            // one set of sums for orders 0..4: F (orders 0..3) and C (1..4)
            expand<0>(acc, F, std::make_integer_sequence<int, 20>{});
            expand<1>(acc + 1, C, std::make_integer_sequence<int, 34>{});
        } else {
            double E[34];
            expand<0>(acc, F, std::make_integer_sequence<int, 20>{});
            expand<1>(acc + 16, E, std::make_integer_sequence<int, 34>{});
            combine_fe(F, E, C, std::make_integer_sequence<int, 34>{});
        }
        const long ab = (long)owner * kSub3 + cell;
        double c[20];
#pragma unroll
        for (int a = 0; a < 20; ++a) c[a] = p.aux[a * p.aux_stride + ab];
        if constexpr (T::source_role)
            scale_inv_fact(c, std::make_integer_sequence<int, 20>{});  // M_b / b!
        double gx[3] = {0.0, 0.0, 0.0};
        grad_x(c, C, gx, std::make_integer_sequence<int, 20>{});
        const long b = p.out_blk ? p.out_blk[owner] : owner;
        const long ob = b * kSub3 + cell;
        if constexpr (T::source_role) {
            scale_inv_fact(F, std::make_integer_sequence<int, 20>{});  // gM_b = F_b / b!
#pragma unroll
            for (int a = 0; a < 20; ++a) p.out0[a * p.out_stride + ob] = F[a];
            if constexpr (T::saved_target) {
                // the target role of the owner's cells, from the sums the
                // forward saved: gX_k += sum_a w_a C'_{a+e_k}
                const int t = p.store_tgt[owner];
                if (t >= 0) {
                    const long tb = (long)t * kSub3 + cell;
                    double Ck[24], Cf[34], w[20];
#pragma unroll
                    for (int k = 0; k < 24; ++k) Ck[k] = p.save[k * p.aux_stride2 + tb];
                    expand<1>(Ck, Cf, std::make_integer_sequence<int, 34>{});
#pragma unroll
                    for (int a = 0; a < 20; ++a) w[a] = p.aux2[a * p.aux_stride2 + tb];
                    double gt[3] = {0.0, 0.0, 0.0};
                    grad_x(w, Cf, gt, std::make_integer_sequence<int, 20>{});
#pragma unroll
                    for (int k = 0; k < 3; ++k) gx[k] += gt[k];
                }
            }
#pragma unroll
            for (int k = 0; k < 3; ++k) p.out1[k * p.out_stride + ob] = gx[k];
        } else {
#pragma unroll
            for (int k = 0; k < 3; ++k) p.out0[k * p.out_stride + ob] += gx[k];
        }
    }
}

// ---------------------------------------------------------------------------
// The source plane in LDS
// ---------------------------------------------------------------------------
// The 64 targets of a z-plane reach 448 of the 576 cells of a source plane:
// the parent criterion cuts half of each corner block away. Rows of 8 to 24
// cells lie one after the other in LDS, a record of 20 doubles (10 units of
// 16 bytes) a cell, odd rows at odd units. A 16-byte read serves 16 lanes per
// cycle, two rows of the mirrored lane pattern: one of even, one of odd y,
// each with 8 cells that differ modulo 8. The even row's units are even and
// cover the even bank groups once, the odd row's the odd ones. Conflicts stay
// all the same: 3.9 cycles an LDS instruction (10.4e9 on 2.67e9 in the forward
// of 32768 sub-grids, 19.6e9 on 4.97e9 with saved sums), where records 22
// doubles apart in freely packed rows had half of the LDS cycles. They do not
// bound the kernel: a copy of it without LDS reads took 1% fewer clocks. 70
// KiB, so two work-groups fit a CU.
constexpr int kPlaneCells = 448;
constexpr int kRecUnits = 10;                             // 16-byte reads of a record
constexpr int kPlaneUnits = kPlaneCells * kRecUnits + kHalo;

struct PlaneTable {
    // staging order: the five whole blocks, then the halves of the corner
    // blocks; unit in LDS | block << 13 | cell of the block's plane << 17 |
    // squared distance of its parent cell from the targets' parents << 23
    uint32_t cell[kPlaneCells];
    int row[kHalo];  // unit of (x, y) in LDS = row[y] + 10 x
    int cells, units;
};

constexpr int parent_gap(int v)
{
    const int q = v / 2;
    return q < 4 ? 4 - q : (q > 7 ? q - 7 : 0);
}

constexpr PlaneTable build_plane_table()
{
    PlaneTable t{};
    int at = 0;
    for (int y = 0; y < kHalo; ++y) {
        bool first = true;
        for (int x = 0; x < kHalo; ++x) {
            if (parent_gap(x) * parent_gap(x) + parent_gap(y) * parent_gap(y) > 16) continue;
            if (first) {
                at += (at + y) & 1;
                t.row[y] = at - kRecUnits * x;
            }
            first = false;
            at += kRecUnits;
        }
    }
    t.units = at;
    constexpr int order[9] = {4, 1, 3, 5, 7, 0, 2, 6, 8};
    int n = 0;
    for (int k = 0; k < 9; ++k)
        for (int c = 0; c < 64; ++c) {
            const int x = 8 * (order[k] % 3) + c % 8, y = 8 * (order[k] / 3) + c / 8;
            const int d2 = parent_gap(x) * parent_gap(x) + parent_gap(y) * parent_gap(y);
            if (d2 > 16) continue;
            t.cell[n++] = (uint32_t)(t.row[y] + kRecUnits * x) | (uint32_t)order[k] << 13 | (uint32_t)c << 17 |
                          (uint32_t)d2 << 23;
        }
    t.cells = n;
    return t;
}
constexpr PlaneTable kPlaneTableHost = build_plane_table();
static_assert(kPlaneTableHost.cells == kPlaneCells && kPlaneTableHost.units <= kPlaneUnits,
              "cells of a source plane in reach");
__constant__ PlaneTable c_plane = build_plane_table();

// Rows of the stencil for the two targets of a z-pair (same parent cell, x
// and y parity 0), per e = source plane - plane of the first: first the
// offsets of both, then those of the first alone, then of the second alone
// (the two differ only where the sphere of near cells does).
struct PairTable {
    uint32_t rows[kMaxRows];
    int range[2 * kReach + 1][4];  // per e + kReach
    int total[3];
};
constexpr PairTable build_pair_table()
{
    PairTable t{};
    int nr = 0;
    for (int e = -kReach; e <= kReach; ++e)
        for (int which = 0; which < 3; ++which) {
            t.range[e + kReach][which] = nr;
            for (int dy = -kReach; dy <= kReach; ++dy)
                for (int dx = -kReach; dx <= kReach;) {
                    int n = 0;
                    for (; dx + n <= kReach; ++n) {
                        const bool a = criterion(8, 8, 8, 8 + dx + n, 8 + dy, 8 + e);
                        const bool b = criterion(8, 8, 9, 8 + dx + n, 8 + dy, 8 + e);
                        if (!(which == 0 ? a && b : which == 1 ? a && !b : b && !a)) break;
                    }
                    if (n > 0) {
                        t.rows[nr++] = pack_row(dy, dx, n);
                        t.total[which] += n;
                        dx += n;
                    } else {
                        ++dx;
                    }
                }
            t.range[e + kReach][which + 1] = nr;
        }
    return t;
}
constexpr PairTable kPairTableHost = build_pair_table();
static_assert(kPairTableHost.total[0] + kPairTableHost.total[1] == 1799 &&
                  kPairTableHost.total[0] + kPairTableHost.total[2] == 1799,
              "stencil size");

// The rows of a plane dealt to the RS wavefronts that share it, which wait for
// each other at the plane's barrier: the longest row left goes to the
// wavefront with the least so far (a row also costs about a quarter of a
// cell); four and more wavefronts take rows of more than 9 cells in pieces.
// Dealt in turn, the busiest wavefronts took 1.14 (RS = 2), 1.20 (RS = 4, pairs
// of targets) and 1.53 (RS = 8) times the mean, summed over the planes; so
// 1.09, 1.07 and 1.20. 4096 sub-grids: forward 13.05 -> 12.52 ms, full
// truncation 24.7 -> 23.6, with saved sums 25.9 -> 25.5; 32 sub-grids (RS = 8)
// 122 -> 114 us.
// KZ = 1: one list a wavefront, for either z parity; KZ = 2: PairTable's three.
template <int KZ, int RS>
struct RowShares {
    static constexpr int kTables = KZ == 1 ? 2 : 1, kLists = KZ == 1 ? 1 : 3;
    uint32_t rows[kTables][kMaxRows];
    int range[kTables][2 * kReach + 1][RS][kLists + 1];
    int cells[kTables][kLists];
};
template <int KZ, int RS>
constexpr RowShares<KZ, RS> build_row_shares()
{
    using R = RowShares<KZ, RS>;
    R t{};
    for (int z = 0; z < R::kTables; ++z) {
        int nr = 0;
        for (int e = 0; e <= 2 * kReach; ++e) {
            uint32_t piece[128] = {};
            int list[128] = {}, cost[128] = {}, owner[128] = {}, n = 0;
            for (int l = 0; l < R::kLists; ++l) {
                const int r0 = KZ == 1 ? kStencilHost.range[z][e][0] : kPairTableHost.range[e][l];
                const int r1 = KZ == 1 ? kStencilHost.range[z][e][1] : kPairTableHost.range[e][l + 1];
                for (int r = r0; r < r1; ++r) {
                    const uint32_t w = KZ == 1 ? kStencilHost.rows[z][r] : kPairTableHost.rows[r];
                    const int dy = (int)(w << 24) >> 24, dx = (int)(w << 16) >> 24, len = (int)(w >> 16);
                    const int cuts = RS == 2 ? 1 : (len + 8) / 9;
                    for (int k = 0; k < cuts; ++k) {
                        const int from = len * k / cuts, to = len * (k + 1) / cuts;
                        piece[n] = pack_row(dy, dx + from, to - from);
                        list[n] = l;
                        cost[n] = 4 * (to - from) * (KZ == 2 && l == 0 ? 2 : 1) + 1;
                        owner[n++] = -1;
                        t.cells[z][l] += to - from;
                    }
                }
            }
            int load[RS] = {};
            for (int done = 0; done < n; ++done) {
                int best = -1, least = 0;
                for (int i = 0; i < n; ++i)
                    if (owner[i] < 0 && (best < 0 || cost[i] > cost[best])) best = i;
                for (int w = 1; w < RS; ++w)
                    if (load[w] < load[least]) least = w;
                owner[best] = least;
                load[least] += cost[best];
            }
            for (int w = 0; w < RS; ++w)
                for (int l = 0; l <= R::kLists; ++l) {
                    t.range[z][e][w][l] = nr;
                    for (int i = 0; l < R::kLists && i < n; ++i)
                        if (owner[i] == w && list[i] == l) t.rows[z][nr++] = piece[i];
                }
        }
    }
    return t;
}
template <int KZ, int RS>
struct RowSharesOf {
    static constexpr RowShares<KZ, RS> host = build_row_shares<KZ, RS>();
    static_assert(KZ == 1 ? host.cells[0][0] == 1799 && host.cells[RowShares<KZ, RS>::kTables - 1][0] == 1799
                          : host.cells[0][0] == kPairTableHost.total[0] &&
                                host.cells[0][RowShares<KZ, RS>::kLists - 2] == kPairTableHost.total[1] &&
                                host.cells[0][RowShares<KZ, RS>::kLists - 1] == kPairTableHost.total[2],
                  "every cell dealt once");
    static_assert(host.range[RowShares<KZ, RS>::kTables - 1][2 * kReach][RS - 1][RowShares<KZ, RS>::kLists] + 1 <=
                      kMaxRows,
                  "a row may be read ahead");
};
template <int KZ, int RS>
__constant__ RowShares<KZ, RS> c_shares = RowSharesOf<KZ, RS>::host;

// A cell of a source plane on its way into LDS: load_cell takes the centre and
// the 20 components from memory (64 lanes read 512 contiguous bytes of a whole
// block) if the cell's parent is within `reach2` (squared) of the targets'
// parents in x and y; put_cell forms the record and writes it with 16-byte LDS
// stores. A missing block is staged far away with zero sources: its terms are
// exact zeros. pk: the cell's table entry.
struct StagedCell {
    double raw[20], x[3];
    int shift;
    bool in, there;
};
template <int MODE>
__device__ __forceinline__ void load_cell(const KParams& p, const int4* s_rel, int zs, int reach2, uint32_t pk,
                                          StagedCell& s)
{
    s.in = (int)(pk >> 23) <= reach2;
    s.there = false;
    if (!s.in) return;
    const int4 rr = s_rel[9 * (zs >> 3) + (int)((pk >> 13) & 15u)];
    if (rr.x < 0) return;
    s.there = true;
    s.shift = rr.z;
    const long o = 64 * (zs & 7) + (int)((pk >> 17) & 63u);
    const double* pm = p.mom + (long)rr.x * kSub3 + o;
    const double* px = p.pos + (long)rr.y * kSub3 + o;
#pragma unroll
    for (int c = 0; c < 20; ++c) s.raw[c] = pm[c * p.mom_stride];
#pragma unroll
    for (int k = 0; k < 3; ++k) s.x[k] = px[k * p.pos_stride];
}
template <int MODE>
__device__ __forceinline__ void put_cell(const KParams& p, const StagedCell& s, uint32_t pk, double2* lds)
{
    using T = ModeTraits<MODE>;
    if (!s.in) return;
    double val[2 * kRecUnits];
    if (s.there) {
#pragma unroll
        for (int k = 0; k < 3; ++k)
            val[k] = s.x[k] + (double)(int)(int8_t)((s.shift >> (8 * k)) & 0xff) * p.period[k];
        stage_record<T::sums, T::source_role>(s.raw, val);
    } else {
#pragma unroll
        for (int k = 0; k < 2 * kRecUnits; ++k) val[k] = k < 3 ? kFar : 0.0;
    }
    double2* dst = lds + (int)(pk & 8191u);
#pragma unroll
    for (int j = 0; j < kRecUnits; ++j) dst[j] = make_double2(val[2 * j], val[2 * j + 1]);
}

// Target planes of a wavefront: two where their sums fit the registers (a
// source record is then read once for both), else one.
template <int MODE>
constexpr int planes_per_wave()
{
    return ModeTraits<MODE>::nacc <= 16 ? 2 : 1;
}
// Wavefronts of a work-group, and the work-list entries of a target: they hold
// KZ planes for each RS wavefronts.
constexpr int group_waves(int rs) { return rs == 8 ? 8 : 4; }
constexpr int parts_per_target(int kz, int rs) { return kSub * rs / (group_waves(rs) * kz); }

// Batched interaction. A work-group takes a part of a target: RS wavefronts
// (lane = x + 8 y) share the same KZ target planes, the stencil rows dealt to
// them, their sums added in order at the end. The source planes in reach of
// the part are staged in LDS one at a time.
//
// RS = 2 and 4: work-groups of 4 wavefronts, two on a CU, so that one's loads
// and barriers are hidden by the other's arithmetic. What bounds it: FP64 issue
// and, above about 80% of it, the power limit (the clock falls from 2.28 GHz at
// 68% to 2.06 at 88%). Sharing rows instead of planes costs more staging (a
// part of 2 planes stages 18 source planes) but no wavefront waits for a
// slower plane at the barriers. 16384 sub-grids with rows dealt in turn, RS =
// 1 / 2 / 4: forward with saved sums 107.9 / 104.9 / 111.4 ms, full truncation
// with saved sums 155.6 / 150.9 / 155.1, forward (two planes a wavefront, so
// a record is read once for both) 57.3 / 53.1 / 52.6, full truncation 113.1 /
// 102.4 / 99.7; with one plane a wavefront the last two took 57.3 and 106.3
// (RS = 2, a slower box). One work-group of 8 or 16 wavefronts a target with
// whole planes of 101 KiB before: forward 55.7, with saved sums 113.5 ms.
//
// RS = 8: one work-group of 8 wavefronts a CU on one target plane, for launches
// that would leave CUs empty or with one work-group. Nothing else hides its
// loads, so two planes are in LDS (141 KiB) and the next one's components come
// into registers while one is worked on: one barrier a plane. 27 targets of an
// open box: 116 us, of it 92 FP64 issue (155 with 4 wavefronts and one plane);
// with saved sums 205 (260). A full chip is better served by two work-groups:
// 4096 sub-grids 15.5 ms against 12.5, with saved sums 28.9 against 26.3.
template <int MODE, int KZ, int RS, bool PERSIST>
__global__ void __launch_bounds__(64 * group_waves(RS), 2) k_interact(const KParams p)
{
    using T = ModeTraits<MODE>;
    constexpr int kThreads = 64 * group_waves(RS);
    constexpr bool kAhead = RS == 8;  // two planes in LDS, the next one's loads in flight
    constexpr int kParts = parts_per_target(KZ, RS);
    constexpr int kPlanes = kSub / kParts;  // target planes of a work-group
    static_assert(RS == 2 || RS == 4 || (RS == 8 && KZ == 1), "wavefronts sharing planes");
    static_assert(T::nc == 2 * kRecUnits, "record size");
    static_assert((KZ == 2 ? RS * KZ : (RS - 1) * (group_waves(RS) / RS)) * T::nacc * 64 <=
                      (kAhead ? 4 : 2) * kPlaneUnits,
                  "merge through the plane");
    __shared__ double2 lds2[(kAhead ? 2 : 1) * kPlaneUnits];
    __shared__ int4 s_rel[27];
    __shared__ int s_row[kHalo];
    __shared__ int s_item, s_step;
    double* lds = reinterpret_cast<double*>(lds2);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int sub = wave % RS;  // share of the rows
    uint32_t pk[2];  // the thread's cells of a plane
    pk[0] = tid < kPlaneCells ? c_plane.cell[tid] : ~0u;
    pk[1] = tid + kThreads < kPlaneCells ? c_plane.cell[tid + kThreads] : ~0u;
    if (tid < kHalo) s_row[tid] = c_plane.row[tid];
    const int xt = lane & 7, yt = lane >> 3;
    const int sgx = (xt & 1) ? -1 : 1;
    const int sgy = (yt & 1) ? -1 : 1;
    const int step_x = sgx * kRecUnits;
    // Persistent launch: the work-group takes work-list entries from a counter
    // until the list is exhausted -- in pieces, from the piece of its XCD
    // (work-group b runs on XCD b mod npieces), then from the following ones
    // until every piece is (s_step: pieces left behind) -- else the one of its
    // index.
    int item = (int)blockIdx.x;
    if (PERSIST && tid == 0) s_step = 0;
#pragma unroll 1
    for (;;) {
        __syncthreads();  // the previous entry is finished by every wavefront
        int index, part;
        if (PERSIST) {
            if (tid == 0) {
                int it = p.n_items;
                const int np = p.npieces > 0 ? p.npieces : 1;
                for (int step = s_step; step < np; ++step) {
                    const int k = ((int)blockIdx.x + step) % np;
                    const int first = p.npieces > 0 ? kParts * p.piece_off[k] : 0;
                    const int count = (p.npieces > 0 ? kParts * p.piece_off[k + 1] : p.n_items) - first;
                    const int i = atomicAdd(p.counter + k, 1);
                    if (i < count) {
                        it = first + i;
                        s_step = step;
                        break;
                    }
                    // every work-group overruns every counter once: the last
                    // to do so leaves it zero for the next launch
                    if (i == count + (int)gridDim.x - 1) atomicExch(p.counter + k, 0);
                    s_step = step + 1;
                }
                s_item = it;
            }
            __syncthreads();
            item = __builtin_amdgcn_readfirstlane(s_item);
            if (item >= p.n_items) break;
            index = item / kParts;  // the parts of a target one after the other: they share their sources
            part = item % kParts;
        } else {
            // a part of every target, then the next: entry i keeps its XCD
            index = item % (p.n_items / kParts);
            part = item / (p.n_items / kParts);
        }
        const int owner = p.order ? p.order[index] : p.first + index;
        if (tid < 27) s_rel[tid] = p.rel[(long)owner * 27 + tid];
        const int z0 = part * kPlanes;                 // first target plane of the work-group
        const int zt = z0 + KZ * (wave / RS);          // of the wavefront
        const int cell = xt + 8 * yt + 64 * zt;
        double xi[KZ], yi[KZ], zi[KZ], acc[KZ * T::nacc];
#pragma unroll
        for (int t = 0; t < KZ; ++t) {
            const long o = (p.own_blk ? p.own_blk[owner] : owner) * (long)kSub3 + cell + 64 * t;
            xi[t] = p.pos[o];
            yi[t] = p.pos[p.pos_stride + o];
            zi[t] = p.pos[2 * p.pos_stride + o];
        }
#pragma unroll
        for (int a = 0; a < KZ * T::nacc; ++a) acc[a] = 0.0;

        // the rows [r0, r1) of a table for the targets T0 .. T1 - 1 of the wavefront
        auto rows = [&](const double2* plane, const uint32_t* table, int r0, int r1, auto t0, auto t1) {
            if (r0 >= r1) return;
            uint32_t w = table[r0];
            int row = s_row[8 + yt + sgy * (int)(int8_t)(w & 0xff)];
            for (int r = r0;;) {
                // the next row's place is read while this one is worked on
                const uint32_t wn = table[r + 1];
                const int next = s_row[8 + yt + sgy * (int)(int8_t)(wn & 0xff)];
                const double2* src = plane + row + kRecUnits * (8 + xt) + step_x * (int)(int8_t)((w >> 8) & 0xff);
                const int n = (int)(w >> 16);
                for (int k = 0; k < n; ++k, src += step_x) {
                    double f[2 * kRecUnits];
#pragma unroll
                    for (int j = 0; j < kRecUnits; ++j) {
                        const double2 v = src[j];
                        f[2 * j] = v.x;
                        f[2 * j + 1] = v.y;
                    }
#pragma unroll
                    for (int t = t0; t < t1; ++t)
                        pair_sums<T::sums>(acc + t * T::nacc, f, xi[t] - f[0], yi[t] - f[1], zi[t] - f[2]);
                }
                if (++r >= r1) break;
                w = wn;
                row = next;
            }
        };

        const int first = 4 + z0 / 2, last = 4 + (z0 + kPlanes - 1) / 2;  // the targets' parent planes
        // the next plane from zs on that can hold a source in reach (a layer of
        // neighbours that are all missing holds none), or -1
        auto plane_from = [&](int zs) {
            while (zs < 2 * (last + 4) + 2) {
                if ((zs & 7) == 0 || zs == 2 * (first - 4)) {
                    bool some = false;
                    for (int b = 0; b < 9; ++b) some |= s_rel[9 * (zs >> 3) + b].x >= 0;
                    if (!some) {
                        zs = (zs | 7) + 1;
                        continue;
                    }
                }
                return zs;
            }
            return -1;
        };
        auto reach2 = [&](int zs) {
            const int ps = zs >> 1;
            const int gap = ps < first ? first - ps : (ps > last ? ps - last : 0);
            return 16 - gap * gap;
        };
        auto add_plane = [&](int zs, const double2* plane) {
            const int e = zs - (8 + zt);
            if (e < -kReach || e > kReach) return;
            constexpr std::integral_constant<int, 0> c0{};
            constexpr std::integral_constant<int, 1> c1{};
            constexpr std::integral_constant<int, KZ> ck{};
            const auto& share = c_shares<KZ, RS>;
            if constexpr (KZ == 1) {
                const int* rg = share.range[zt & 1][e + kReach][sub];
                rows(plane, share.rows[zt & 1], rg[0], rg[1], c0, c1);
            } else {
                const int* rg = share.range[0][e + kReach][sub];
                rows(plane, share.rows[0], rg[0], rg[1], c0, ck);
                rows(plane, share.rows[0], rg[1], rg[2], c0, c1);
                rows(plane, share.rows[0], rg[2], rg[3], c1, ck);
            }
        };
        __syncthreads();  // s_rel is there
        if constexpr (kAhead) {
            int zs = plane_from(2 * (first - 4));
            StagedCell ahead;
            if (zs >= 0) load_cell<MODE>(p, s_rel, zs, reach2(zs), pk[0], ahead);
            double2* plane = lds2;
            while (zs >= 0) {
                put_cell<MODE>(p, ahead, pk[0], plane);
                const int next = plane_from(zs + 1);
                if (next >= 0) load_cell<MODE>(p, s_rel, next, reach2(next), pk[0], ahead);
                // every wavefront is past the plane before, whose buffer is written next
                __syncthreads();
                add_plane(zs, plane);
                plane = plane == lds2 ? lds2 + kPlaneUnits : lds2;
                zs = next;
            }
        } else {
#pragma unroll 1
            for (int zs = plane_from(2 * (first - 4)); zs >= 0; zs = plane_from(zs + 1)) {
                __syncthreads();  // the previous plane is no longer read
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    StagedCell c;
                    load_cell<MODE>(p, s_rel, zs, reach2(zs), pk[it], c);
                    put_cell<MODE>(p, c, pk[it], lds2);
                }
                __syncthreads();
                add_plane(zs, lds2);
            }
        }

        // the sums of the wavefronts that share planes are added in their order
        __syncthreads();  // the last plane is no longer read
        if constexpr (KZ == 2) {
            // all four share: each of the first two finishes a plane
            static_assert(RS == 4, "four wavefronts a pair of planes");
#pragma unroll
            for (int a = 0; a < KZ * T::nacc; ++a) lds[(sub * KZ * T::nacc + a) * 64 + lane] = acc[a];
            __syncthreads();
            if (sub < KZ) {
                const double* from = lds + sub * T::nacc * 64 + lane;
                double sum[T::nacc];
#pragma unroll
                for (int a = 0; a < T::nacc; ++a) {
                    sum[a] = from[a * 64];
#pragma unroll
                    for (int w = 1; w < RS; ++w) sum[a] += from[(w * KZ * T::nacc + a) * 64];
                }
                store_sums<MODE>(p, owner, cell + 64 * sub, sum);
            }
        } else if constexpr (RS == 8) {
            // the eighth of the sums that each wavefront adds up, then the first
            if (sub > 0) {
#pragma unroll
                for (int a = 0; a < T::nacc; ++a) lds[((sub - 1) * T::nacc + a) * 64 + lane] = acc[a];
            }
            __syncthreads();
            for (int a = sub; a < T::nacc; a += RS) {
                double v = lds[a * 64 + lane];
#pragma unroll
                for (int w = 1; w < RS - 1; ++w) v += lds[(w * T::nacc + a) * 64 + lane];
                lds[a * 64 + lane] = v;
            }
            __syncthreads();
            if (sub == 0) {
#pragma unroll
                for (int a = 0; a < T::nacc; ++a) acc[a] += lds[a * 64 + lane];
                store_sums<MODE>(p, owner, cell, acc);
            }
        } else {
            double* mine = lds + (wave / RS) * (RS - 1) * T::nacc * 64;
            if (sub > 0) {
#pragma unroll
                for (int a = 0; a < T::nacc; ++a) mine[((sub - 1) * T::nacc + a) * 64 + lane] = acc[a];
            }
            __syncthreads();
            if (sub == 0) {
#pragma unroll
                for (int a = 0; a < T::nacc; ++a) {
#pragma unroll
                    for (int w = 0; w < RS - 1; ++w) acc[a] += mine[(w * T::nacc + a) * 64 + lane];
                    if (a % 4 == 3) __builtin_amdgcn_sched_barrier(0);  // few loads in flight: the registers are full
                }
                store_sums<MODE>(p, owner, cell, acc);
            }
        }
        if (!PERSIST) break;
    }
}

}  // namespace
