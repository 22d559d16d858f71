// chain.h -- the Eq. 5-6 recurrence of one column spread over the waves of a
// workgroup, for launches with fewer columns than the chip can hold (one
// frame, a few frames): what bounds those is the chain row -> row, so the
// chain is given a wave of its own and everything that does not depend on a
// cost is taken out of it.
//
// With data(b, k) = PO[f][k+1] - PO[f][b], f = f(b, k) the rounded mean of
// rows b..k, a candidate of row k costs
//     min(C_o + T_oo [+ c_ord if f > f_prev + tau], C_s + T_so) + data
//     or C_g + T_go [+ c_grav / c_dive by f] + data,
// where only C_o, C_g, C_s and f_prev (row b-1) belong to the chain.  Roles:
//   wave 0        the chain.  Lane l holds the row k = l mod 64 of the window
//                 (j, j+64] above the current row j: step j reads row j's
//                 result from its lane, folds the stixels that start at
//                 b = j+1 into the 64 rows of the window and hands the lane
//                 to row j+64.  Its operands (data, the ground penalty, f)
//                 come out of an LDS ring.
//   waves 1, 2    "prep": fill the ring, up to kRing groups ahead.
//   wave 4        summaries of finished groups, for the far waves' test.
//   the others    "far": a wave takes one 64-row slot and one parity of base
//                 groups at a time and folds the stixels longer than 64 rows
//                 (and b = 0) into the slot's rows, in base order, as the
//                 chain publishes them.  Such a stixel's base lies 64 or more
//                 steps behind the row it ends at, so these waves may lag the
//                 chain by most of a slot before it waits for them.
// Steps go in groups of eight; a group is handed over by one LDS flag.
//
// What bounds it: the chain wave's own instructions, about 27 a step and 210
// cycles with the hand-overs (a step of dp_kernel<7, 2, 1> took 920: its wave
// also tabulated the prior over the means and folded every open slot).
// Measured, one road scene a launch, the whole kernel against dp_kernel with
// one wave per column: 640x240 83 -> 31 us, 1024x440 165 -> 51, 1280x720 with
// 7-pixel columns 961 -> 76, 2048x880 with 256 disparities 1454 -> 144 (409
// columns on 256 compute units, two to a unit: there the far waves bound it).
//
// Waits: the chain at group G waits for prep of group G and for the far
// candidates of its rows, which need the base groups up to G-8; prep of group g
// waits for the chain's group g-kRing; far group g waits for the chain's group
// g, its test for group g+kFarLag of an earlier slot, and a far wave's tasks
// ascend.  Every wait is for a smaller group, so all end; each is bounded all
// the same (kSpinLimit polls, then the column is given up and reported with
// overflow 255).
//
// Ties: far candidates of a row have smaller bases than the window's, so a
// window candidate replaces one only when strictly smaller, and within each
// the bases ascend: the first candidate in Eq. 6's order wins, as in
// dp_column.h.  Costs on the grid only (sums are exact, in any order).
#pragma once

#include "dp_column.h"

namespace stx {

constexpr int kGroup = 8;          // steps per hand-over
constexpr int kRing = 4;           // groups in the prep ring
constexpr int kChainWaves = 16;    // most waves per column
constexpr int kPrepWaves = 2;
constexpr int kSpinLimit = 1 << 22;

// Rows the chain's arrays hold: the chain runs whole pairs of groups.
__host__ __device__ constexpr int chain_rows(int H) { return (H + 15) & ~15; }
// Waves of a column of H rows, at most `most`: 0 the chain, 1 and 2 prep, 4 the
// summaries (columns of more than two slots), the others far.  Waves go to the
// four SIMDs in turn, and no far wave is put on the chain's (0, 4, 8, 12: a
// far wave beside the chain was half as fast, and the chain waited for it).
__host__ __device__ constexpr int chain_waves(int H, int most) {
    const int far = 2 * ((H + 63) / 64 - 1);          // tasks beyond the first slot's
    int n = 4;                                        // waves 3, 5, 6, 7, 9, 10, 11, ... are far
    for (int have = 1; have < far && n < most; ++n) have += (n & 3) != 0;
    return n;
}

// Workgroups of `waves` waves and `lds` bytes (their static part included) that
// a compute unit of gfx950 holds: 16 waves, the kernels taking up to 128
// registers a lane, and 160 KB of LDS in blocks of 1,280 bytes.
__host__ __device__ constexpr int chain_resident(int waves, int lds) {
    const int by_lds = 160 * 1024 / ((lds + 1279) / 1280 * 1280), by_waves = 16 / waves;
    return by_lds < by_waves ? by_lds : by_waves;
}

struct ChainFlags {
    int prep[kRing];               // group held by a ring place, plus one
    int done;                      // groups the chain has finished
    int summed;                    // groups whose summary is written
    int far[kMaxSlots][2];         // row groups of a slot whose far candidates are in, by
                                   // the parity of their base groups
    int abort;
    int pad;
};

// Blocks of rows in the bound on a far stixel's data cost.  (Blocks of 16
// rows keep 0.21 of the far groups of a road scene instead of 0.27, for four
// times the bounds.)
constexpr int kBlock = 32;
constexpr int kBoundStride = kMaxHeight / kBlock + 1;   // block boundaries
static_assert(edge_row_floats(kBlock) == 2, "entries 32 i of the table");

// LDS of one column, laid out by its height (bytes; every part 16-aligned):
// per base b {PA, PN2, diving, gravity threshold} and {PG, PS, PM, unused}; per
// row the published {C_o, f << 16 | b, C_g, C_s} (before that the far candidates'
// {cost, f << 16 | b}: those of even base groups in its first two words, of odd
// ones in the other two); the ring, {data, data +
// ground prior, f << 16 | b, pixel's ground / sky cost} per step and lane; the
// bounds; the groups' summaries; the flags.
struct ChainLds {
    float4* base;                  // [H+1]
    float4* pre;                   // [H+1]
    float4* rec;                   // [rows]
    float4* ring;                  // [kRing * kGroup][64]
    float* bound;                  // [33][33]
    float4* sum;                   // [rows / 8] summaries of groups
    ChainFlags* fl;
};
constexpr int kBoundBytes = (kBoundStride * kBoundStride * 4 + 15) & ~15;
__host__ __device__ constexpr size_t chain_lds_bytes(int H) {
    return (size_t)((H + 1) * 32 + chain_rows(H) * 18 + kRing * kGroup * 64 * 16 + kBoundBytes +
                    (int)sizeof(ChainFlags));
}
__device__ __forceinline__ ChainLds chain_lds(char* p, int H) {
    ChainLds L;
    const int R = chain_rows(H);
    L.base = reinterpret_cast<float4*>(p);
    L.pre = L.base + (H + 1);
    L.ring = L.pre + (H + 1);
    L.rec = L.ring + kRing * kGroup * 64;
    L.bound = reinterpret_cast<float*>(L.rec + R);
    L.sum = reinterpret_cast<float4*>(reinterpret_cast<char*>(L.bound) + kBoundBytes);
    L.fl = reinterpret_cast<ChainFlags*>(L.sum + R / kGroup);
    return L;
}

// Keeps LDS accesses of the two sides apart for the compiler; the LDS itself
// serves a wave's accesses in order.
__device__ __forceinline__ void lds_order() { asm volatile("" ::: "memory"); }
typedef volatile __attribute__((address_space(3))) int LdsFlag;   // read and written in LDS, as such
__device__ __forceinline__ int flag_peek(const int* p) { return *(LdsFlag*)p; }
__device__ __forceinline__ int flag_read(const int* p) {
    return __builtin_amdgcn_readfirstlane(flag_peek(p));
}
__device__ __forceinline__ void flag_write(int* p, int v) {
    lds_order();
    if ((threadIdx.x & 63) == 0) *(LdsFlag*)p = v;
    lds_order();
}
// Waits until *p >= want; false when the column is given up.
__device__ __forceinline__ bool flag_wait(const int* p, int want, ChainFlags* fl,
                                          int* got = nullptr) {
    int v;
    for (int n = 0; (v = flag_read(p)) < want; ++n) {
        if ((n & 3) != 3) continue;
        if (n >= kSpinLimit || flag_read(&fl->abort)) {
            flag_write(&fl->abort, 1);
            return false;
        }
        __builtin_amdgcn_s_sleep(1);
    }
    if (got) *got = v;
    lds_order();
    return true;
}

// x of another lane of the same eight, within the instruction that reads it.
template <int CTRL>
__device__ __forceinline__ float quad(float x) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
        0, __builtin_bit_cast(int, x), CTRL, 0xf, 0xf, true));
}

// A column as the chain's waves see it.
struct ChainCol {
    int H, vtop, fbase, nrow;
    uint32_t stride4;              // bytes between rows of the object prefix table
    __amdgpu_buffer_rsrc_t po;
    float eps;
    float T00, T00c, T10, T20, c_grav, c_dive;   // T00c = T00 + the ordering penalty
    __device__ __forceinline__ float at(uint32_t off) const { return buf_load_b(po, off, 0u); }
};

// The cost-independent part of the stixels [b, k] for one base b (uniform)
// and the lane's row: mean f, gathers of PO[f][k+1] and PO[f][b] and the
// ground predecessor's prior.
struct ChainPair {
    float dk, db, pg;
    int pk;
};
template <bool GR>
__device__ __forceinline__ ChainPair chain_pair(const ChainCol& c, const float4 bs, const int b,
                                                const float eA, const float eN,
                                                const uint32_t koff) {
    ChainPair r;
    const int f = mean_index(eA - bs.x, eN - bs.y, c.eps);
    r.dk = c.at(__umul24((uint32_t)f, c.stride4) + koff);
    r.db = c.at(__umul24((uint32_t)f, c.stride4) +
                ((uint32_t)(b * 4) - (uint32_t)c.fbase * c.stride4));
    r.pk = (f << 16) | b;
    r.pg = 0.0f;
    if constexpr (GR) {
        const float lo = (f < __builtin_bit_cast(int, bs.w)) ? c.c_grav : 0.0f;
        r.pg = ((f > __builtin_bit_cast(int, bs.z)) ? c.c_dive : lo) + c.T10;
    }
    return r;
}

// A row's best object stixel is kept as f << 16 | b.  A stixel {f, b} pays the
// ordering penalty over a predecessor {f', b'}, b' < b, iff f > f' + tau, that
// is iff (f << 16 | b) - chain_ord >= (f' << 16 | b').
__device__ __forceinline__ int chain_ord(const Prior& P) {
    return (min(P.tau_ord, 256) + 1) << 16;
}

// What the far waves' test needs of a finished group of steps: with A(b) the
// cheapest prior and predecessor of base b, min over its bases of A(b) - PM[b],
// and C_g - PG, C_s - PS after its last row.
__device__ __forceinline__ void chain_summary(const ChainCol& c, const ChainLds& L, const int G) {
    const int lane = threadIdx.x & 63;
    const int j = G * kGroup + (lane & 7);            // < 64 (slots - 1) < H
    const float4 r = L.rec[j], p = L.pre[j + 1];
    float lb = vmin(vmin(r.x + c.T00, r.z + c.T10), r.w + c.T20) - p.z;
    lb = vmin(lb, quad<0xB1>(lb));                    // lanes 1,0,3,2
    lb = vmin(lb, quad<0x4E>(lb));                    // lanes 2,3,0,1
    lb = vmin(lb, quad<0x141>(lb));                   // the other half of eight
    if (lane == 7) L.sum[G] = make_float4(lb, r.z - p.x, r.w - p.y, 0.0f);
    flag_write(&L.fl->summed, G + 1);
}

// Prep wave p of np: the ring entries of groups p, p + np, ...
__device__ __forceinline__ void chain_prep(const ChainCol& c, const ChainLds& L, const int p,
                                           const int np) {
    const int lane = threadIdx.x & 63;
    const int ngroups = chain_rows(c.H) / kGroup;
    for (int g = p; g < ngroups; g += np) {
        const int j0 = g * kGroup, jl0 = j0 & 63, s0 = j0 & ~63;
        // the lane's row in this slot and in the next
        const int k0 = min(s0 + lane, c.H - 1), k1 = min(s0 + 64 + lane, c.H - 1);
        const float4 e0 = L.base[k0 + 1], e1 = L.base[k1 + 1];
        const uint32_t fb = (uint32_t)c.fbase * c.stride4;
        const uint32_t o0 = (uint32_t)(k0 + 1) * 4u - fb, o1 = (uint32_t)(k1 + 1) * 4u - fb;
        ChainPair r[kGroup];
        float4 bs[kGroup];                            // read together: one LDS latency
#pragma unroll
        for (int u = 0; u < kGroup; ++u) bs[u] = L.base[min(j0 + u + 1, c.H - 1)];
        auto pairs = [&](auto GR) {
#pragma unroll
            for (int u = 0; u < kGroup; ++u) {
                const bool up = lane <= jl0 + u;      // the lane has moved on to the next slot
                const int b = min(j0 + u + 1, c.H - 1);
                r[u] = chain_pair<decltype(GR)::value>(c, bs[u], b, up ? e1.x : e0.x,
                                                       up ? e1.y : e0.y, up ? o1 : o0);
            }
        };
        // above vtop no ground stixel precedes (C_g is INF there)
        if (j0 <= c.vtop) pairs(std::true_type{});
        else pairs(std::false_type{});
        // each row's ground (even lanes; INF above vtop) or sky cost
        float ec[kGroup], pp[kGroup + 1];
#pragma unroll
        for (int u = 0; u <= kGroup; ++u)
            pp[u] = reinterpret_cast<const float*>(L.pre + min(j0 + u, c.H))[lane & 1];
#pragma unroll
        for (int u = 0; u < kGroup; ++u)
            ec[u] = ((lane & 1) || j0 + u <= c.vtop) ? pp[u + 1] - pp[u] : inf_f();
        if (g >= kRing && !flag_wait(&L.fl->done, g - kRing + 1, L.fl)) return;
        const int at = (g & (kRing - 1)) * kGroup * 64 + lane;
#pragma unroll
        for (int u = 0; u < kGroup; ++u) {
            const float d = r[u].dk - r[u].db;
            L.ring[at + 64 * u] =
                make_float4(d, d + r[u].pg, __builtin_bit_cast(float, r[u].pk), ec[u]);
        }
        flag_write(&L.fl->prep[g & (kRing - 1)], g + 1);
    }
}

// The column's prefixes at block boundaries, while the bounds are made: rows of
// 4 (H / 128 + 1) floats in LDS, in the ring's and the records' place (both
// unused yet).
__device__ __forceinline__ int chain_edge_quads(int H) { return H / kBlock / 4 + 1; }
__device__ __forceinline__ float* chain_edges(const ChainLds& L) {
    return reinterpret_cast<float*>(L.ring);
}

// Stages them from the table of entries 32 i (rows of edge_row_floats(H)).
__device__ __forceinline__ void chain_load_edges(const ChainCol& c, const ChainLds& L,
                                                 const float* edge, const int wave, const int nw) {
    const int lane = threadIdx.x & 63;
    const int nb = c.H / kBlock, nq = chain_edge_quads(c.H), row = edge_row_floats(c.H);
    float* const tile = chain_edges(L);
    const auto er = make_rsrc(edge, (uint32_t)(c.nrow * row) * 4u);
    const uint32_t off = (uint32_t)min(lane, nb) * 4u;
    constexpr int U = 8;
    for (int f0 = wave; f0 < c.nrow; f0 += U * nw) {
        float x[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            x[u] = buf_load_b(er, off, (uint32_t)(min(f0 + u * nw, c.nrow - 1) * row) * 4u);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (lane < 4 * nq && f0 + u * nw < c.nrow) tile[(f0 + u * nw) * 4 * nq + lane] = x[u];
    }
}

// bound[i][j] = min over f of the object cost of rows [i B, j B) at mean f (no
// stixel costs those rows less) from the staged edges.  A lane takes one i and
// four neighbouring j, a wave 64 such lanes and a part of the means; the parts'
// minima meet in LDS (bound holds +inf before).
__device__ __forceinline__ void chain_bounds(const ChainCol& c, const ChainLds& L, const int wave,
                                             const int nw) {
    const int lane = threadIdx.x & 63;
    const int nb = c.H / kBlock, nq = chain_edge_quads(c.H);
    const float* const tile = chain_edges(L);
    const int items = (nb + 1) * nq, sets = (items + 63) >> 6, parts = max(nw / sets, 1);
    for (int w = wave; w < sets * parts; w += nw) {
        const int set = w % sets, part = w / sets;
        const int it = min(set * 64 + lane, items - 1), i = it / nq, q = it - i * nq;
        float v0 = inf_f(), v1 = v0, v2 = v0, v3 = v0;
#pragma unroll 4
        for (int f = part; f < c.nrow; f += parts) {
            const float a = tile[f * 4 * nq + i];
            const float4 x = reinterpret_cast<const float4*>(tile)[f * nq + q];
            v0 = vmin(v0, x.x - a);
            v1 = vmin(v1, x.y - a);
            v2 = vmin(v2, x.z - a);
            v3 = vmin(v3, x.w - a);
        }
        const float v[4] = {v0, v1, v2, v3};
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (set * 64 + lane < items && 4 * q + t >= i && 4 * q + t <= nb)
                __hip_atomic_fetch_min(&L.bound[i * kBoundStride + 4 * q + t], v[t],
                                       __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }
}

// Far wave: rows of slot s, the bottom stixel and of the bases 1 .. 64 s those
// whose group of eight has parity par.  Below the slot's neighbour a group is skipped when no
// row of the slot can use it: with A(b) the cheapest prior and predecessor of
// base b, every stixel [b, k] costs at least
//     A(b) + PM[iB] - PM[b] + bound[i][j] + PM[k+1] - PM[jB]
// (iB and jB the block boundaries inside [b, k], PM the prefix of each pixel's
// smallest object cost over all means), and OB^k is at most
//     U(k) = min(candidates so far,
//                C_g(j) + PG[k] - PG[j+1] + T_go + max penalty + own
//                    (above vtop: ground to vtop, then sky to k-1),
//                C_s(j) + PS[k] - PS[j+1] + T_so + own),
// j the last row of a group kFarLag later, own the largest cost of a pixel
// that is an object stixel of its own.  A group whose bounds all exceed U(k)
// holds no candidate of the minimum, nor a tie with it.  On road scenes three
// of four groups go this way; a column of one long object keeps most of them.
constexpr int kFarLag = 4;
__device__ __forceinline__ bool chain_far(const ChainCol& c, const ChainLds& L, const Prior& P,
                                          const int s, const int par) {
    const int lane = threadIdx.x & 63;
    const int k = min(64 * s + lane, c.H - 1);
    const float4 e = L.base[k + 1];
    const uint32_t koff = (uint32_t)(k + 1) * 4u - (uint32_t)c.fbase * c.stride4;
    float m;
    int pk;
    {
        const int f = mean_index(e.x, e.y, c.eps);
        m = c.at(__umul24((uint32_t)f, c.stride4) + koff) + P.first[0];
        pk = f << 16;
    }
    // the result of rows [8 i0, 8 i1) of the slot, and its flag (only those
    // rows: the chain may already have finished earlier ones)
    auto publish = [&](int i0, int i1) {
        if ((lane >> 3) >= i0 && (lane >> 3) < i1 && 64 * s + lane < chain_rows(c.H))
            reinterpret_cast<float2*>(L.rec + 64 * s + lane)[par] =
                make_float2(m, __builtin_bit_cast(float, pk));
        flag_write(&L.fl->far[s][par], i1);
    };
    if (s == 0) {
        publish(0, 8);
        return true;
    }
    const int kord = chain_ord(P);
    const float T20 = c.T20;
    // row k's parts of U and of the bound
    const float4 p0 = L.pre[k], p1 = L.pre[k + 1];
    const float4 pv = L.pre[max(min(c.vtop + 1, c.H), 0)];
    const float ug = ((k - 1 <= c.vtop)
        ? p0.x + c.T10 + __builtin_fmaxf(c.c_grav, c.c_dive)
        : pv.x + P.trans[1][2] + (p0.y - pv.y) + T20) + P.own_max;
    const float us = p0.y + T20 + P.own_max;
    const int jb = (k + 1) / kBlock;
    const float wk = p1.z - L.pre[jb * kBlock].z;
    const int ng = 8 * s, near = 8 * (s - 1);
    float w = 0.0f;
    int done = 0, summed = 0;                         // as last read
    ChainPair ra[kGroup], rb[kGroup];
    // whether any row may use group g (waits for the rows its test reads)
    auto test = [&](int g, bool& use) -> bool {
        use = true;
        if (g >= near) return true;                   // the slot below: nearly always of use
        if ((g & 3) == par) {                         // the first of its block
            const int i = g * kGroup / kBlock + 1;
            w = L.pre[i * kBlock].z + L.bound[i * kBoundStride + jb] + wk;
        }
        const int gl = min(g + kFarLag, near - 1);
        if (summed <= gl && !flag_wait(&L.fl->summed, gl + 1, L.fl, &summed)) return false;
        const float lb = L.sum[g].x;
        const float4 sl = L.sum[gl];
        const float U = vmin(vmin(m, sl.y + ug), sl.z + us);
        use = __ballot(lb + w <= U) != 0;
        return true;
    };
    // a group's cost-independent part (the wave-uniform operands are read
    // together: one LDS latency)
    auto gather = [&](ChainPair (&r)[kGroup], int g) {
        float4 bs[kGroup];
#pragma unroll
        for (int u = 0; u < kGroup; ++u) bs[u] = L.base[8 * g + 1 + u];
        // above vtop no ground stixel precedes (C_g is INF there)
        if (8 * g <= c.vtop) {
#pragma unroll
            for (int u = 0; u < kGroup; ++u)
                r[u] = chain_pair<true>(c, bs[u], 8 * g + 1 + u, e.x, e.y, koff);
        } else {
#pragma unroll
            for (int u = 0; u < kGroup; ++u)
                r[u] = chain_pair<false>(c, bs[u], 8 * g + 1 + u, e.x, e.y, koff);
        }
    };
    auto finish = [&](const ChainPair (&r)[kGroup], int g, bool use) -> bool {
        if (use) {
            if (done <= g && !flag_wait(&L.fl->done, g + 1, L.fl, &done)) return false;
            float4 o[kGroup];                         // rows b-1
#pragma unroll
            for (int u = 0; u < kGroup; ++u) o[u] = L.rec[8 * g + u];
#pragma unroll
            for (int u = 0; u < kGroup; ++u) {
                const float pen =
                    (r[u].pk - kord >= __builtin_bit_cast(int, o[u].y)) ? c.T00c : c.T00;
                // C_g is INF above vtop
                const float x = vmin(vmin(o[u].x + pen, o[u].w + T20), o[u].z + r[u].pg) +
                                (r[u].dk - r[u].db);
                const bool better = x < m;
                m = better ? x : m;
                pk = better ? r[u].pk : pk;
            }
        }
        // with near group i folded, rows 8 i .. have every far base of this
        // parity, and so have the eight rows after them
        const int i = g - near;
        if (i >= 0) publish(i, min(i + 2, 8));
        return true;
    };
    // a group's gathers are in flight while the one before it is folded
    bool ua = false, ub = false;
    if (!test(par, ua)) return false;
    if (ua) gather(ra, par);
    for (int g = par; g < ng; g += 4) {               // 4 s groups of a parity
        if (par && g == near + 1) publish(0, 1);      // rows 0 .. 7 need no odd near group
        if (!test(g + 2, ub)) return false;
        if (ub) gather(rb, g + 2);
        if (!finish(ra, g, ua)) return false;
        ua = false;
        if (g + 4 < ng && !test(g + 4, ua)) return false;
        if (ua) gather(ra, g + 4);
        if (!finish(rb, g + 2, ub)) return false;
    }
    return true;
}

// The chain (wave 0).  Returns false when the column is given up.  The ground
// and sky costs share a register: even lanes hold C_g, odd lanes C_s (a quad
// permutation hands either to every lane, or swaps them, within the
// instruction that reads it).
__device__ __forceinline__ bool chain_run(const ChainCol& c, const ChainLds& L, const Prior& P) {
    constexpr int kGround = 0xA0, kSky = 0xF5, kSwap = 0xB1;   // quad_perm 0,0,2,2 1,1,3,3 1,0,3,2
    const int lane = threadIdx.x & 63;
    const int ngroups = chain_rows(c.H) / kGroup;
    const bool odd = lane & 1;
    const float INF = inf_f();
    float T00 = c.T00, T00c = c.T00c, T20 = P.trans[2][0];
    asm("" : "+v"(T00), "+v"(T00c), "+v"(T20));   // vector registers: operands beside a scalar or a permuted one
    const float tO = odd ? P.trans[0][2] : P.trans[0][1];      // object -> this lane's class
    const float tX = odd ? P.trans[1][2] : P.trans[2][1];      // the other class -> this one
    const int kord = chain_ord(P);
    // the operands of the eight steps ahead of each step
    float4 o[kGroup];
    auto fetch = [&](int u, int G) {
        o[u] = L.ring[((G % kRing) * kGroup + u) * 64 + lane];
    };
    // flags of a group and the far candidates they guard (read in this order)
    int fprep, ffar0, ffar1;
    float4 far;
    auto peek = [&](int G) {
        fprep = flag_peek(&L.fl->prep[(G + 1) % kRing]);
        ffar0 = flag_peek(&L.fl->far[G >> 3][0]);
        ffar1 = flag_peek(&L.fl->far[G >> 3][1]);
        lds_order();
        far = L.rec[min((G * kGroup & ~63) + lane, chain_rows(c.H) - 1)];
    };
    float m = INF, C = odd ? P.first[2] : P.first[1];
    int pk = 0;
    if (!flag_wait(&L.fl->prep[0], 1, L.fl)) return false;
#pragma unroll
    for (int u = 0; u < kGroup; ++u) fetch(u, 0);
    peek(0);
    __builtin_amdgcn_s_waitcnt(0xc07f);   // as in the loop's slow way in
#pragma unroll 1
    for (int G = 0; G < ngroups; ++G) {
        // this group's far candidates and the next group's operands are there
        const int want = (G + 1 < ngroups) ? G + 2 : 0;
        auto ready = [&]() {
            return __builtin_amdgcn_readfirstlane(fprep) >= want &&
                   __builtin_amdgcn_readfirstlane(min(ffar0, ffar1)) >= (G & 7) + 1;
        };
        if (!ready()) {
            // no sleep between polls: everything else waits for this wave
            int n = 0;
            do {
                if (++n > kSpinLimit || ((n & 255) == 0 && flag_read(&L.fl->abort))) {
                    flag_write(&L.fl->abort, 1);
                    return false;
                }
                peek(G);
                // nothing is in flight past here: the other way to the group's
                // first uses then decides how long those wait
                __builtin_amdgcn_s_waitcnt(0xc07f);
            } while (!ready());
        }
        const int j0 = G * kGroup, jl0 = j0 & 63, Gn = min(G + 1, ngroups - 1);
        {   // the group's rows take in their far candidates: the cheaper of the
            // two parities', on a tie the smaller base, and on a tie with the
            // window's again the far one (its base is smaller)
            const int q0 = __builtin_bit_cast(int, far.y), q1 = __builtin_bit_cast(int, far.w);
            const bool second = far.z < far.x || (far.z == far.x && (q1 & 0xffff) < (q0 & 0xffff));
            const float fm = second ? far.z : far.x;
            const bool take = ((lane >> 3) == (jl0 >> 3)) && fm <= m;
            m = take ? fm : m;
            pk = take ? (second ? q1 : q0) : pk;
        }
        peek(Gn);
        float hC = 0.0f;
        int hm = 0, hp = 0;
#pragma unroll
        for (int u = 0; u < kGroup; ++u) {
            const int jl = jl0 + u;
            C += o[u].w;                                         // row j's ground and sky costs
            const float Co = readlane_f(m, jl);
            const int pj = readlane_i(pk, jl);
            hC = ((lane >> 1) == u) ? C : hC;
            asm("v_writelane_b32 %0, %1, %2" : "+v"(hm) : "s"(Co), "n"(u));
            asm("v_writelane_b32 %0, %1, %2" : "+v"(hp) : "s"(pj), "n"(u));
            // the stixels that start at j+1; lane jl goes on to row j+64: its
            // cost becomes a NaN, which any candidate replaces
            asm("v_writelane_b32 %0, -1, %1" : "+v"(m) : "s"(jl));
            const int p = __builtin_bit_cast(int, o[u].z);
            const float pen = (p - kord >= pj) ? T00c : T00;
            const float t = vmin(Co + pen, quad<kSky>(C) + T20);
            const float x = vmin(t + o[u].x, quad<kGround>(C) + o[u].y);
            const bool better = !(x >= m);
            m = better ? x : m;
            pk = better ? p : pk;
            // running minima for row j+1: T_gg and T_ss are >= 0, so staying
            // in a class never costs more than a new stixel of it
            C = vmin(vmin(Co + tO, quad<kSwap>(C) + tX), C);
            // the step's operands make room for the next group's: a load issued
            // before their last use would go to other registers, and be waited
            // for to be copied at the loop's end
            asm volatile("" : "+v"(m), "+v"(pk) :: "memory");
            fetch(u, Gn);
        }
        if (lane < 8)
            *reinterpret_cast<float2*>(L.rec + j0 + lane) =
                make_float2(__builtin_bit_cast(float, hm), __builtin_bit_cast(float, hp));
        if (lane < 16) reinterpret_cast<float*>(L.rec + j0 + (lane >> 1))[2 + (lane & 1)] = hC;
        flag_write(&L.fl->done, G + 1);
    }
    return true;
}

// Backtracking from the published rows (wave 0).  An object stixel's base and
// mean are stored with its row; a ground or sky stixel starts at the last
// base at which a new stixel was strictly cheaper than the running minimum.
// The predecessor is the first class (object, ground, sky) that attains the
// candidate's minimum.
__device__ __forceinline__ void chain_backtrack(const ChainCol& c, const ChainLds& L,
                                                const Prior& P, const ColumnOut& out) {
    const int lane = threadIdx.x & 63;
    const int ktop = c.H - 1;
    auto row = [&](int p, float& Co, float& Cg, float& Cs, int& pk) {
        const float4 r = L.rec[p];
        Co = r.x;
        pk = __builtin_bit_cast(int, r.y);
        Cg = r.z;
        Cs = r.w;
    };
    float tO, tG, tS;
    int tp;
    row(ktop, tO, tG, tS, tp);
    float total = tO;
    int ctop = 0;
    if (tG < total) { total = tG; ctop = 1; }
    if (tS < total) { total = tS; ctop = 2; }
    ctop = __builtin_amdgcn_readfirstlane(ctop);
    auto walk = [&](bool direct, int n_total, RecRegs& rr) -> int {
        int k = ktop, cls = ctop, t = 0;
        float target = total;
        while (true) {
            int b = 0, f = 0;
            if (cls == 0) {
                const int pk = __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, L.rec[k].y));
                b = pk & 0xffff;
                f = pk >> 16;
            } else {
                // last j < k with a strictly cheaper new stixel at b = j+1
                for (int j0 = (k - 1) & ~63; j0 >= 0 && k > 0; j0 -= 64) {
                    const int j = j0 + lane;
                    bool imp = false;
                    if (j < k) {
                        float Co, Cg, Cs;
                        int pk;
                        row(j, Co, Cg, Cs, pk);
                        imp = (cls == 1)
                            ? vmin(Co + P.trans[0][1], Cs + P.trans[2][1]) < Cg && j + 1 <= c.vtop
                            : vmin(Co + P.trans[0][2], Cg + P.trans[1][2]) < Cs;
                    }
                    const uint64_t mk = __ballot(imp);
                    if (mk) {
                        b = j0 + (63 - __builtin_clzll(mk)) + 1;
                        break;
                    }
                }
            }
            int cp = -1;
            float prevC = 0.0f;
            if (b > 0) {
                float Co, Cg, Cs;
                int pkp;
                row(b - 1, Co, Cg, Cs, pkp);
                float x0, x1, x2;
                if (cls == 0) {
                    const float4 bs = L.base[b];
                    x0 = Co + P.trans[0][0] + ((f > (pkp >> 16) + P.tau_ord) ? P.c_ord : 0.0f);
                    const float lo = (f < __builtin_bit_cast(int, bs.w)) ? P.c_grav : 0.0f;
                    x1 = Cg + P.trans[1][0] +
                         ((f > __builtin_bit_cast(int, bs.z)) ? P.c_dive : lo);
                    x2 = Cs + P.trans[2][0];
                } else if (cls == 1) {
                    x0 = Co + P.trans[0][1];
                    x1 = Cg + P.trans[1][1];
                    x2 = Cs + P.trans[2][1];
                } else {
                    x0 = Co + P.trans[0][2];
                    x1 = Cg + P.trans[1][2];
                    x2 = Cs + P.trans[2][2];
                }
                const float mn = vmin(vmin(x0, x1), x2);
                cp = (x0 == mn) ? 0 : ((x1 == mn) ? 1 : 2);
                cp = __builtin_amdgcn_readfirstlane(cp);
                prevC = pick3(Co, Cg, Cs, cp);
            }
            const float cost = (b > 0) ? target - prevC : target;
            if (!direct) {
                if (lane == t) pack_record(b, k, cls, f, cost, rr.w0, rr.w1, rr.w2);
            } else {
                const int pos = n_total - 1 - t;
                if (pos < out.cap && lane == 0) {
                    uint32_t w0, w1;
                    float w2;
                    pack_record(b, k, cls, f, cost, w0, w1, w2);
                    out.rec[pos * 3 + 0] = w0;
                    out.rec[pos * 3 + 1] = w1;
                    out.rec[pos * 3 + 2] = __builtin_bit_cast(uint32_t, w2);
                }
            }
            ++t;
            if (b == 0 || t > c.H) break;
            k = b - 1;
            cls = cp;
            target = prevC;
        }
        return t;
    };
    RecRegs rr{0u, 0u, 0.0f};
    const int n = walk(false, 0, rr);
    if (n <= 64) {
        const int pos = n - 1 - lane;
        if (lane < n && pos < out.cap) {
            out.rec[pos * 3 + 0] = rr.w0;
            out.rec[pos * 3 + 1] = rr.w1;
            out.rec[pos * 3 + 2] = __builtin_bit_cast(uint32_t, rr.w2);
        }
    } else {
        RecRegs dummy{0u, 0u, 0.0f};
        walk(true, n, dummy);
    }
    if (lane == 0) {
        *out.count = n < out.cap ? n : out.cap;
        *out.total = total;
        *out.overflow = (uint8_t)(n > out.cap ? 1 : 0);
    }
}

// A column for the chain's waves: its object prefix table (rows of stride4
// bytes, row f - fbase) and constants.
__device__ __forceinline__ ChainCol chain_column(const int H, const int vtop, const Prior& P,
                                                 const float* PO, const int fbase, const int fmax,
                                                 const uint32_t stride4) {
    ChainCol c;
    c.H = H;
    c.vtop = vtop;
    c.fbase = fbase;
    c.nrow = fmax - fbase + 1;
    c.stride4 = stride4;
    c.po = make_rsrc(PO, (uint32_t)c.nrow * stride4);
    c.eps = P.mean_eps;
    c.T00 = P.trans[0][0];
    c.T00c = P.trans[0][0] + P.c_ord;
    c.T10 = P.trans[1][0];
    c.T20 = P.trans[2][0];
    c.c_grav = P.c_grav;
    c.c_dive = P.c_dive;
    return c;
}

// Clears the flags and bounds (by every thread, ahead of a barrier).
__device__ __forceinline__ void chain_clear(const ChainLds& L) {
    if (threadIdx.x < sizeof(ChainFlags) / 4) reinterpret_cast<int*>(L.fl)[threadIdx.x] = 0;
    for (int i = threadIdx.x; i < kBoundStride * kBoundStride; i += (int)blockDim.x)
        L.bound[i] = inf_f();
}

// One column by the whole workgroup (chain_waves(H, ..) waves), its base, pre
// and bound arrays filled and its flags cleared.  Results are written by wave
// 0, to where get_out() says then; the LDS may be reused after a barrier.
template <class Out>
__device__ __forceinline__ void chain_solve(const ChainCol& c, const ChainLds& L, const Prior& P,
                                            Out&& get_out) {
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int nw = (int)(blockDim.x >> 6);
    const int slots = (c.H + 63) >> 6;
    if (wave == 0) {
        __builtin_amdgcn_s_setprio(3);
        const bool ok = chain_run(c, L, P);
        __builtin_amdgcn_s_setprio(0);
        const ColumnOut out = get_out();
        if (ok) {
            chain_backtrack(c, L, P, out);
        } else if (lane == 0) {
            *out.count = 0;
            *out.total = inf_f();
            *out.overflow = 255;
        }
    } else if (wave <= kPrepWaves) {
        chain_prep(c, L, wave - 1, kPrepWaves);
    } else if (wave == 4) {
        // the groups that far waves test
        for (int g = 0; g < 8 * (slots - 2); ++g) {
            if (!flag_wait(&L.fl->done, g + 1, L.fl)) break;
            chain_summary(c, L, g);
        }
    } else if ((wave & 3) != 0) {
        const int nf = nw - 3 - ((nw - 1) >> 2), f = wave - 3 - (wave >> 2);
        // tasks in turn: slot 0 (bottom stixels only), then of each slot the
        // even and the odd base groups, so that the nearest slots are always
        // being worked on
        bool ok = true;
        for (int t = f; ok && t < 2 * slots; t += nf) ok = chain_far(c, L, P, t >> 1, t & 1);
    }
}

// One column from its prefix tables in memory (in).  lds: 16-byte aligned,
// chain_lds_bytes(H).
__device__ __forceinline__ void solve_chain(const int H, const int vtop, const Prior& P,
                                            const ColumnIn& in, const ColumnOut& out, char* lds) {
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int nw = (int)(blockDim.x >> 6);
    const ChainLds L = chain_lds(lds, H);
    const ChainCol c = chain_column(H, vtop, P, in.PO, in.fbase, in.fmax,
                                    (uint32_t)in.po_stride * 4u);
    chain_clear(L);
    for (int b = threadIdx.x; b <= H; b += (int)blockDim.x) {
        const int r = max(H - 1 - b, 0);
        L.base[b] = make_float4(in.PA[b], in.PN2[b], __builtin_bit_cast(float, in.fg_hi[r]),
                                __builtin_bit_cast(float, in.fg_lo[r]));
        L.pre[b] = make_float4(in.PG[b], in.PS[b], in.PM[b], 0.0f);
    }
    if (H > 64) {
        chain_load_edges(c, L, in.PO_edge, wave, nw);
        __syncthreads();
        chain_bounds(c, L, wave, nw);
    }
    __syncthreads();
    chain_solve(c, L, P, [&]() { return out; });
}

}  // namespace stx
