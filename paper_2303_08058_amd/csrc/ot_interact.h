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
    int range[2][2 * kReach + 1][3];      // per (pz, dz+9): first row, split row, end row
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
            // split point: first row at which the running count reaches half
            int split = first, run = 0;
            while (split < nr && 2 * run < offs) {
                run += (int)(t.rows[pz][split] >> 16);
                ++split;
            }
            if (split > first && 2 * run - offs > offs - 2 * (run - (int)(t.rows[pz][split - 1] >> 16)))
                --split;
            t.range[pz][dz + kReach][0] = first;
            t.range[pz][dz + kReach][1] = split;
            t.range[pz][dz + kReach][2] = nr;
            total += offs;
        }
        t.count[pz] = total;
    }
    return t;
}

constexpr StencilTable kStencilHost = build_stencil();
static_assert(kStencilHost.count[0] == 1799 && kStencilHost.count[1] == 1799, "stencil size");
__constant__ StencilTable c_stencil = build_stencil();

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
            for (int r = rg[0]; r < rg[2]; ++r) {
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
    const int* order;      // work-group -> owner (NULL: identity)
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
    double period[3];
    int* counter;          // persistent launch: work counter(s), zeroed before the launch
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

// LDS plane layout: cell-major, Layout::stride doubles per cell -- the
// source record (stage_record of ot_pair.h), then padding. A pair is read with
// 16-byte loads from one base address (immediate offsets).
// The cell stride in 16-byte units is odd, so the 8 lanes served per LDS
// cycle by a 16-byte read -- 8 different cells modulo 8 in the mirrored lane
// pattern -- fall on disjoint banks.
template <int MODE>
struct Layout {
    static constexpr int nc = ModeTraits<MODE>::nc;
    static constexpr int nvec = (nc + 1) / 2;                               // 16-byte reads per cell
    static constexpr int stride = (nvec % 2 == 1) ? 2 * nvec : 2 * nvec + 2;  // doubles per cell
};

template <int MODE, int NW, int NP>
constexpr int lds_doubles()
{
    constexpr int plane = Layout<MODE>::stride * kPlane;
    constexpr int merge = (NW == 16 || NP == 2) ? 20 * kSub3 : 0;
    return plane > merge ? plane : merge;
}

// Staging of one source z-plane (the 24 x 24 cells of the 3 x 3 neighbour
// blocks), one cell per thread: thread v takes cell v & 63 of block v >> 6
// (the block is wavefront-uniform, so its relation is a scalar load), loads
// the cell's centre and each of its moments once (a load of a wavefront reads
// 512 contiguous bytes), forms the source record with
// compile-time factors, and writes the cell's record with 16-byte LDS
// stores. A missing neighbour block is staged far away with zero sources.
template <int MODE, int NW>
__device__ __forceinline__ void stage_plane(const KParams& p, const int4* rel, int zs, int tid, double* lds)
{
    using T = ModeTraits<MODE>;
    using Lay = Layout<MODE>;
    for (int v = tid; v < 9 * 64; v += NW * 64) {
        const int bxy = __builtin_amdgcn_readfirstlane(v >> 6);
        const int lane = v & 63;
        const int by = bxy / 3, bx = bxy - 3 * by;
        const int4 rr = rel[9 * (zs >> 3) + bxy];  // uniform address: scalar load
        const bool present = rr.x >= 0;
        const long o = 64 * (zs & 7) + lane;
        const double* pm = p.mom + (present ? (long)rr.x * kSub3 : 0) + o;
        const double* px = p.pos + (present ? (long)rr.y * kSub3 : 0) + o;
        const long sm = p.mom_stride, sx = p.pos_stride;
        double sh[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) sh[k] = (double)(int)(int8_t)((rr.z >> (8 * k)) & 0xff) * p.period[k];
        double val[2 * Lay::nvec];
#pragma unroll
        for (int c = 0; c < 2 * Lay::nvec; ++c) val[c] = 0.0;
        if (present) {
            double raw[20];
#pragma unroll
            for (int c = 0; c < 20; ++c) raw[c] = pm[c * sm];
#pragma unroll
            for (int k = 0; k < 3; ++k) val[k] = px[k * sx] + sh[k];
            stage_record<T::sums, T::source_role>(raw, val);
        } else {
#pragma unroll
            for (int k = 0; k < 3; ++k) val[k] = kFar;
        }
        double2* dst = reinterpret_cast<double2*>(
            lds + ((by * 8 + (lane >> 3)) * kHalo + bx * 8 + (lane & 7)) * Lay::stride);
#pragma unroll
        for (int j = 0; j < Lay::nvec; ++j) dst[j] = make_double2(val[2 * j], val[2 * j + 1]);
    }
}

// NP = 2 (8 wavefronts): two passes over the source planes, target planes
// 0-3 then 4-7, two wavefronts per target plane with its stencil rows split
// in halves as with 16 wavefronts. Each pass stages the 21 source planes in
// its reach (42 instead of 24), and in exchange the work per staged plane is
// spread evenly over the 4 SIMDs (about 95% against 86% for one pass with a
// wavefront per target plane).
template <int MODE, int NW, int NP, bool PERSIST>
__global__ void __launch_bounds__(NW * 64) k_interact(const KParams p)
{
    using T = ModeTraits<MODE>;
    using Lay = Layout<MODE>;
    static_assert(NW == 8 || NW == 16, "8 or 16 wavefronts");
    static_assert(NP == 1 || (NP == 2 && NW == 8), "two passes: 8 wavefronts");
    constexpr bool HALVES = NW == 16 || NP == 2;  // two wavefronts per target plane
    __shared__ double lds[lds_doubles<MODE, NW, NP>()];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half = HALVES ? (wave & 1) : 0;
    // Persistent launch (counter != NULL): the work-group takes work-list
    // entries from a global counter until the list is exhausted; otherwise it
    // does the one entry of its index.
    __shared__ int s_item;
    constexpr bool persistent = PERSIST;
    int item = (int)blockIdx.x;
    // in pieces: the work-group starts on the piece of its XCD (work-group b
    // runs on XCD b mod npieces) and moves on to the next piece when that is
    // exhausted, until every piece is (s_step: pieces left behind)
    __shared__ int s_step;
    if (persistent && tid == 0) s_step = 0;
#pragma unroll 1
    for (;;) {
    if (persistent) {
        __syncthreads();  // the previous entry is finished by every wavefront
        if (tid == 0) {
            int it = p.n_items;
            if (p.npieces > 0) {
                for (int step = s_step; step < p.npieces; ++step) {
                    const int k = ((int)blockIdx.x + step) % p.npieces;
                    const int i = atomicAdd(p.counter + k, 1);
                    if (i < p.piece_off[k + 1] - p.piece_off[k]) {
                        it = p.piece_off[k] + i;
                        s_step = step;
                        break;
                    }
                }
            } else {
                it = atomicAdd(p.counter, 1);
            }
            s_item = it;
        }
        __syncthreads();
        item = __builtin_amdgcn_readfirstlane(s_item);
        if (item >= p.n_items) break;
    }
    const int owner = p.order ? p.order[item] : item;
    const int4* s_rel = p.rel + (long)owner * 27;  // this owner's relations
#pragma unroll 1
    for (int pass = 0; pass < NP; ++pass) {
    // With 8 wavefronts and one pass (wave w on SIMD w % 4) the target planes
    // are paired per SIMD as (0,4) (1,6) (2,5) (3,7): the pairing whose summed
    // per-plane work varies least from one staged plane to the next.
    const int zt = (NW == 16) ? (wave >> 1)
                 : (NP == 2) ? 4 * pass + (wave >> 1)
                             : (wave == 5 ? 6 : (wave == 6 ? 5 : wave));
    const int xt = lane & 7, yt = lane >> 3;
    const int pz = zt & 1;
    const int cell = xt + 8 * yt + 64 * zt;
    const int sgx = (xt & 1) ? -1 : 1;
    const int sgy = (yt & 1) ? -1 : 1;

    double xi, yi, zi;
    {
        const long b = p.own_blk ? p.own_blk[owner] : owner;
        const long o = b * kSub3 + cell;
        xi = p.pos[o];
        yi = p.pos[p.pos_stride + o];
        zi = p.pos[2 * p.pos_stride + o];
    }

    double acc[T::nacc];
#pragma unroll
    for (int a = 0; a < T::nacc; ++a) acc[a] = 0.0;

    // addresses in 16-byte units of the LDS plane
    constexpr int cs = Lay::stride / 2;
    const int lane_off = ((8 + yt) * kHalo + 8 + xt) * cs;
    const int step_x = sgx * cs;
    const int step_y = sgy * kHalo * cs;
    const double2* lds2 = reinterpret_cast<const double2*>(lds);

    const int zs_begin = NP == 2 ? (pass == 0 ? 0 : 8 + 4 - kReach) : 0;
    const int zs_end = NP == 2 ? (pass == 0 ? 8 + 3 + kReach + 1 : kHalo) : kHalo;
    for (int zs = zs_begin; zs < zs_end; ++zs) {
        __syncthreads();
        stage_plane<MODE, NW>(p, s_rel, zs, tid, lds);
        __syncthreads();
        const int dz = zs - (8 + zt);
        if (dz >= -kReach && dz <= kReach) {
            const int* rg = c_stencil.range[pz][dz + kReach];
            int r0 = rg[0], r1 = rg[2];
            if (HALVES) {
                if (half == 0)
                    r1 = rg[1];
                else
                    r0 = rg[1];
            }
            for (int r = r0; r < r1; ++r) {
                const uint32_t w = c_stencil.rows[pz][r];
                const int dy = (int)(int8_t)(w & 0xff);
                const int dx0 = (int)(int8_t)((w >> 8) & 0xff);
                const int n = (int)(w >> 16);
                int off = lane_off + dy * step_y + dx0 * step_x;
                for (int k = 0; k < n; ++k, off += step_x) {
                    double f[2 * Lay::nvec];
#pragma unroll
                    for (int j = 0; j < Lay::nvec; ++j) {
                        const double2 v = lds2[off + j];
                        f[2 * j] = v.x;
                        f[2 * j + 1] = v.y;
                    }
                    pair_sums<T::sums>(acc, f, xi - f[0], yi - f[1], zi - f[2]);
                }
            }
        }
    }

    // ---------------- epilogues ----------------
    if constexpr (HALVES) {
        // the two wavefronts of a target plane add their partial sums, through
        // LDS in rounds of at most 20 components
#pragma unroll
        for (int a0 = 0; a0 < T::nacc; a0 += 20) {
            __syncthreads();
            if (half == 1) {
#pragma unroll
                for (int a = a0; a < T::nacc && a < a0 + 20; ++a) lds[(a - a0) * kSub3 + cell] = acc[a];
            }
            __syncthreads();
            if (half == 0) {
#pragma unroll
                for (int a = a0; a < T::nacc && a < a0 + 20; ++a) acc[a] += lds[(a - a0) * kSub3 + cell];
            }
        }
        if (half == 1) continue;  // the next pass (none after the last)
    }
    store_sums<MODE>(p, owner, cell, acc);
    }  // pass
    if (!persistent) break;
    }  // work-list entries
}

// zeroes the kMaxPieces counters of a persistent launch (one per lane)
__global__ void k_zero_counter(int* c) { c[threadIdx.x] = 0; }

}  // namespace
