// ot_cells.h -- the interaction of few targets: a work-group per one or two
// target cells, its threads spread over the cells' sources. Included by
// ot_fmm.hip after ot_interact.h (stencil criterion, relations, epilogues).
#pragma once

#include "ot_interact.h"

namespace {

// Sources of a group of KT target cells, from the criterion: for KT = 1 the
// offsets from a target of parity (0, 0, 0); for KT = 2 the offsets from the
// first of the two cells of an x pair (x parity 0 and 1, y and z parity 0),
// with the cells of the pair they belong to. Packed dx | dy << 8 | dz << 16 |
// cells << 24, x fastest. Other parities mirror the axis (KT = 2: y and z).
template <int KT>
constexpr int count_cell_sources()
{
    int n = 0;
    for (int dz = -kReach; dz <= kReach; ++dz)
        for (int dy = -kReach; dy <= kReach; ++dy)
            for (int dx = -kReach; dx <= kReach; ++dx)
                n += criterion(8, 8, 8, 8 + dx, 8 + dy, 8 + dz) ||
                     (KT == 2 && criterion(9, 8, 8, 8 + dx, 8 + dy, 8 + dz));
    return n;
}
template <int KT>
struct CellSources {
    static constexpr int n = count_cell_sources<KT>();
    uint32_t at[n];
};
template <int KT>
constexpr CellSources<KT> build_cell_sources()
{
    CellSources<KT> t{};
    int n = 0;
    for (int dz = -kReach; dz <= kReach; ++dz)
        for (int dy = -kReach; dy <= kReach; ++dy)
            for (int dx = -kReach; dx <= kReach; ++dx) {
                const uint32_t first = criterion(8, 8, 8, 8 + dx, 8 + dy, 8 + dz) ? 1u : 0u;
                const uint32_t second = (KT == 2 && criterion(9, 8, 8, 8 + dx, 8 + dy, 8 + dz)) ? 2u : 0u;
                if (first | second)
                    t.at[n++] = (uint32_t)(dx & 0xff) | (uint32_t)(dy & 0xff) << 8 | (uint32_t)(dz & 0xff) << 16 |
                                (first | second) << 24;
            }
    return t;
}
static_assert(CellSources<1>::n == 1799, "stencil size");
template <int KT>
__constant__ CellSources<KT> c_cell_sources = build_cell_sources<KT>();

// Target cells of a work-group: two where their accumulators (2 x 16) leave
// room for a source's record and the pair step below 256 registers.
template <int MODE>
constexpr int cells_per_group()
{
    return ModeTraits<MODE>::nacc <= 16 ? 2 : 1;
}

// v of the lane whose number differs in BIT (8), or in BIT and all lower bits
// (4, 2, 1): one DPP move.
template <int BIT>
__device__ __forceinline__ double lane_pair(double v)
{
    constexpr int kCtrl = BIT == 8 ? 0x128 : BIT == 4 ? 0x141 : BIT == 2 ? 0x1b : 0xb1;
    int2 w = __builtin_bit_cast(int2, v);
    w.x = __builtin_amdgcn_mov_dpp(w.x, kCtrl, 0xf, 0xf, true);
    w.y = __builtin_amdgcn_mov_dpp(w.y, kCtrl, 0xf, 0xf, true);
    return __builtin_bit_cast(double, w);
}

// Exchanges a's upper with b's lower half of every 2 BIT lanes (BIT 32, 16).
template <int BIT>
__device__ __forceinline__ void swap_halves(double& a, double& b)
{
    const uint2 x = __builtin_bit_cast(uint2, a), y = __builtin_bit_cast(uint2, b);
    uint2 u, w;
    if constexpr (BIT == 32) {
        const auto lo = __builtin_amdgcn_permlane32_swap(x.x, y.x, false, false);
        const auto hi = __builtin_amdgcn_permlane32_swap(x.y, y.y, false, false);
        u = make_uint2(lo[0], hi[0]);
        w = make_uint2(lo[1], hi[1]);
    } else {
        const auto lo = __builtin_amdgcn_permlane16_swap(x.x, y.x, false, false);
        const auto hi = __builtin_amdgcn_permlane16_swap(x.y, y.y, false, false);
        u = make_uint2(lo[0], hi[0]);
        w = make_uint2(lo[1], hi[1]);
    }
    a = __builtin_bit_cast(double, u);
    b = __builtin_bit_cast(double, w);
}

// Adds v[0 .. N) over the 64 lanes of a wavefront: each step hands half of
// the values to a lane whose number differs in BIT and keeps the other half,
// so N values cost about N exchanges instead of 6 N. Returns the index whose
// sum this lane ends up with, in v[0], or -1. The order of the additions is
// fixed.
template <int N, int BIT>
__device__ __forceinline__ int lanes_sum(double* v, int lane, int base, int count)
{
    if constexpr (BIT == 0) {
        return count > 0 ? base : -1;
    } else {
        constexpr int H = (N + 1) / 2;
        const bool up = (lane & BIT) != 0;
#pragma unroll
        for (int i = 0; i < H; ++i) {
            double lo = v[i], hi = i + H < N ? v[i + H] : 0.0;
            if constexpr (BIT >= 16) {
                swap_halves<BIT>(lo, hi);
                v[i] = lo + hi;
            } else {
                v[i] = (up ? hi : lo) + lane_pair<BIT>(up ? lo : hi);
            }
        }
        base += up ? H : 0;
        count = up ? count - H : (count < H ? count : H);
        return lanes_sum<H, BIT / 2>(v, lane, base, count);
    }
}

// One work-group of NT threads per KT target cells. A launch over few targets
// leaves most of the chip idle when a work-group owns a plane of cells; here a
// single sub-grid is 256 or 512 work-groups, each thread takes a few sources
// (4 of NT = 512) straight from memory (a source serves both cells of a pair),
// and the partial sums meet by lane exchange and once through LDS. Work-groups
// go to the XCDs in turn: each takes one z-plane of cells of every target, so
// that an L2 holds the 18 source planes in reach instead of all 24 (64 blocks
// as futures on 16 streams 737 us, 800 with the cells dealt in turn). One
// sub-grid, forward: 8 us (145 with k_interact); with saved sums 11 (156); of
// 18, 4.7 and 9.3 each. What bounds it then is the L1 (rows of up to 18 cells
// of 23 components, read once a work-group) and the list and the merge, about
// half of the instructions (k_interact on a full chip takes 3.1 us: a staged
// source serves 64 or 128 targets there).
template <int MODE, int KT, int NT>
__global__ void __launch_bounds__(NT, NT == 512 ? 2 : 3) k_cells(const KParams p)
{
    using T = ModeTraits<MODE>;
    constexpr int kGroups = kSub3 / KT;
    constexpr int kWaves = NT / 64;
    constexpr int kN = KT * T::nacc;
    __shared__ double s_sum[kWaves][kN];
    __shared__ int4 s_rel[27];
    const int tid = threadIdx.x;
    const int owner = p.first + (int)blockIdx.x / kGroups;
    const int g = (int)(blockIdx.x & 7u) * (kGroups / 8) + (((int)blockIdx.x % kGroups) >> 3);
    const int cell0 = KT * g;  // the group's first cell; a pair shares x / 2, y, z
    const int xt = cell0 & 7, yt = (cell0 >> 3) & 7, zt = cell0 >> 6;
    // halo place hx | hy << 8 | hz << 16 | cells << 24 of a list entry
    auto place = [&](uint32_t w) {
        const int dx = (int)(int8_t)(w & 0xff), dy = (int)(int8_t)((w >> 8) & 0xff),
                  dz = (int)(int8_t)((w >> 16) & 0xff);
        return (uint32_t)(8 + xt + (KT == 1 && (xt & 1) ? -dx : dx)) |
               (uint32_t)(8 + yt + ((yt & 1) ? -dy : dy)) << 8 | (uint32_t)(8 + zt + ((zt & 1) ? -dz : dz)) << 16 |
               (w & 0xff000000u);
    };
    // Batched: the entries whose block is there are gathered in list order, so
    // that no thread is given a missing source (27 targets of an open box,
    // a third of the sources missing: 164 us with the missing ones skipped in
    // turn).
    constexpr int kList = CellSources<KT>::n;
    __shared__ uint32_t s_list[T::halo ? 1 : kList];
    int n = kList;
    if constexpr (!T::halo) {
        __shared__ int s_count[kWaves];
        if (tid < 27) s_rel[tid] = p.rel[(long)owner * 27 + tid];
        __syncthreads();
        constexpr int kEach = (kList + NT - 1) / NT;  // consecutive entries of a thread
        uint32_t mine[kEach];
        uint32_t there = 0;
#pragma unroll
        for (int k = 0; k < kEach; ++k) {
            const int i = tid * kEach + k;
            mine[k] = place(c_cell_sources<KT>.at[i < kList ? i : 0]);
            const int slot = (int)((mine[k] >> 3) & 31u) + 3 * (int)((mine[k] >> 11) & 31u) +
                             9 * (int)((mine[k] >> 19) & 31u);
            if (i < kList && s_rel[slot].x >= 0) there |= 1u << k;
        }
        // the thread's first entry comes after those of the lanes and wavefronts before it
        const int had = __popc(there);
        int at = had;
        for (int d = 1; d < 64; d <<= 1) {
            const int v = __shfl_up(at, d);
            at += (tid & 63) >= d ? v : 0;
        }
        if ((tid & 63) == 63) s_count[tid >> 6] = at;
        at -= had;
        __syncthreads();
        n = 0;
        for (int w = 0; w < kWaves; ++w) {
            at += w < (tid >> 6) ? s_count[w] : 0;
            n += s_count[w];
        }
#pragma unroll
        for (int k = 0; k < kEach; ++k)
            if ((there >> k) & 1u) s_list[at++] = mine[k];
        __syncthreads();
    }
    double xi[KT], yi[KT], zi[KT];
#pragma unroll
    for (int t = 0; t < KT; ++t) {
        const long o = T::halo ? (8 + xt + t) + kHalo * (8 + yt) + kPlane * (8 + zt)
                               : (p.own_blk ? p.own_blk[owner] : owner) * (long)kSub3 + cell0 + t;
        xi[t] = p.pos[o];
        yi[t] = p.pos[p.pos_stride + o];
        zi[t] = p.pos[2 * p.pos_stride + o];
    }
    double acc[kN];
#pragma unroll
    for (int a = 0; a < kN; ++a) acc[a] = 0.0;
    for (int i = tid; i < n; i += NT) {
        uint32_t h;
        if constexpr (T::halo)
            h = place(c_cell_sources<KT>.at[i]);
        else
            h = s_list[i];
        const int hx = (int)(h & 0xff), hy = (int)((h >> 8) & 0xff), hz = (int)((h >> 16) & 0xff);
        long om, ox;
        double sh[3] = {0.0, 0.0, 0.0};
        if constexpr (T::halo) {
            om = ox = hx + kHalo * hy + kPlane * hz;
        } else {
            const int4 rr = s_rel[(hx >> 3) + 3 * (hy >> 3) + 9 * (hz >> 3)];
            const int c = (hx & 7) + 8 * (hy & 7) + 64 * (hz & 7);
            om = (long)rr.x * kSub3 + c;
            ox = (long)rr.y * kSub3 + c;
#pragma unroll
            for (int k = 0; k < 3; ++k) sh[k] = (double)(int)(int8_t)((rr.z >> (8 * k)) & 0xff) * p.period[k];
        }
        constexpr int nm = T::sums == SUMS_MONO ? 1 : 20;
        double raw[nm], rec[T::nc];
#pragma unroll
        for (int c = 0; c < nm; ++c) raw[c] = p.mom[c * p.mom_stride + om];
#pragma unroll
        for (int k = 0; k < 3; ++k) rec[k] = p.pos[k * p.pos_stride + ox] + sh[k];
        stage_record<T::sums, T::source_role>(raw, rec);
#pragma unroll
        for (int t = 0; t < KT; ++t)
            if (KT == 1 || ((h >> (24 + t)) & 1u))
                pair_sums<T::sums>(acc + t * T::nacc, rec, xi[t] - rec[0], yi[t] - rec[1], zi[t] - rec[2]);
    }
    const int mine = lanes_sum<kN, 32>(acc, tid & 63, 0, kN);
    if (mine >= 0) s_sum[tid >> 6][mine] = acc[0];
    __syncthreads();
    if (tid < kN) {
        double v = s_sum[0][tid];
        for (int w = 1; w < kWaves; ++w) v += s_sum[w][tid];
        s_sum[0][tid] = v;
    }
    __syncthreads();
    // one thread per target cell finishes
    if (tid < KT) {
        double sum[T::nacc];
#pragma unroll
        for (int a = 0; a < T::nacc; ++a) sum[a] = s_sum[0][tid * T::nacc + a];
        store_sums<MODE>(p, owner, cell0 + tid, sum);
    }
}

}  // namespace
