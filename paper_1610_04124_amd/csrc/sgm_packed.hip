// sgm_packed.hip -- the path passes of semi-global matching (sgm.hip) with
// path costs in bytes, for penalties that keep them there.
//
// A path cost L_r(p, d) is at most C + P2 (its minimum term is at most M + P2,
// and M is subtracted), so with P2 <= 193 it fits a byte.  Directions write a
// plane of bytes [frame][y][x][d] each, side by side in one launch since none
// needs another.  Where there are many lines, three do (top-down, bottom-up,
// right to left), and the left-to-right pass reads the planes, adds its own
// costs in registers, selects and checks: 6 bytes of memory traffic per pixel
// and disparity where 16-bit sums that the passes added to in turn took 12.
// Where there are few, all four do, and a selection with a workgroup per row
// reads them: a row's steps then stand once in the chain of a call, not twice.
//
// With many lines the vector ALU bounds it, so the costs of two disparities
// share a register (16 bits each, packed instructions): a lane holds 2 R
// disparities, a line LPL lanes (2 R LPL >= D), a wave 64 / LPL lines.  Kept
// relative to the last step's minimum, a step is
//     t = C + min(L, min(L(d-1), L(d+1)) + P1, P2),  L = t - min over d of t
// (t is the path cost).  With eight disparities to a lane and 16 lanes to a line
// that is 74 instructions for 512 disparities (90 us of a pair against 212):
// 32 + 4 of them the Hamming costs, 6 the minimum over the line, which four
// disparities to a lane pay for 256.  With few lines the chain of a row's steps
// bounds it, and the Hamming costs go to a second wave (row_pair_pass).
// 1024x440, 128 disparities, before (one disparity per register, four launches
// over 16-bit sums) and now: one pair 888 / 179 us, 64 pairs 13.56 / 5.71 ms,
// of these 3.3 the three directions (11 GB written), 2.2 the last one and the
// selection (11 GB read, 5 TB/s), 0.3 the census.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "internal.h"
#include "sgm.h"

namespace stx::sgm {

namespace {

constexpr int kCostOut = 62;        // cost of a disparity that leaves the image
constexpr uint32_t kPast = 0x40004000u;   // cost of disparities past D: never a minimum

typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u16x2 h2(uint32_t x) { return __builtin_bit_cast(u16x2, x); }
__device__ __forceinline__ uint32_t w2(u16x2 x) { return __builtin_bit_cast(uint32_t, x); }
__device__ __forceinline__ uint32_t pk_min(uint32_t a, uint32_t b) {
    return w2(__builtin_elementwise_min(h2(a), h2(b)));
}
// Minimum of three, on whole numbers below 0x7c00: as half floats these are the
// positive ones without infinity and NaN, in the same order (and denormals are
// kept), so the half floats' three-way minimum does for them.
__device__ __forceinline__ uint32_t pk_min3(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t r;
    asm("v_pk_minimum3_f16 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
__device__ __forceinline__ uint32_t pk_add(uint32_t a, uint32_t b) { return w2(h2(a) + h2(b)); }
__device__ __forceinline__ uint32_t pk_sub(uint32_t a, uint32_t b) { return w2(h2(a) - h2(b)); }

// Set bits of x, added to acc: the instruction's own addend, which a sum of
// three terms isn't taken apart for.
__device__ __forceinline__ uint32_t bit_count(uint32_t x, uint32_t acc) {
    uint32_t r;
    asm("v_bcnt_u32_b32 %0, %1, %2" : "=v"(r) : "v"(x), "v"(acc));
    return r;
}

template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t old, uint32_t x) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)x, CTRL, 0xf, 0xf, false);
}

// The lane below's and the lane above's value within a line; all ones at the
// line's ends (edge: all ones in the line's first / last lane, else zero).  A
// disparity has a neighbour on one side at least, so the smaller of the two is
// always a cost.
template <int LPL>
__device__ __forceinline__ uint32_t from_below(uint32_t x, uint32_t edge) {
    if constexpr (LPL == 16) return dpp<0x111>(~0u, x);            // row_shr:1
    const uint32_t v = dpp<0x138>(~0u, x);                         // wave_shr:1
    return LPL == 64 ? v : (v | edge);
}
template <int LPL>
__device__ __forceinline__ uint32_t from_above(uint32_t x, uint32_t edge) {
    if constexpr (LPL == 16) return dpp<0x101>(~0u, x);            // row_shl:1
    const uint32_t v = dpp<0x130>(~0u, x);                         // wave_shl:1
    return LPL == 64 ? v : (v | edge);
}

// Value of lane u of each row of 16 lanes, in all of it.
template <int U>
__device__ __forceinline__ uint64_t row_word(uint64_t x) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)x, 0x150 + U, 0xf, 0xf, true);
    const uint32_t hi =
        (uint32_t)__builtin_amdgcn_mov_dpp((int)(uint32_t)(x >> 32), 0x150 + U, 0xf, 0xf, true);
    return ((uint64_t)hi << 32) | lo;
}

// Minimum over a line's lanes, in every lane of it.
template <int LPL>
__device__ __forceinline__ uint32_t line_min(uint32_t x) {
    x = min(x, dpp<0xB1>(~0u, x));                                 // quad_perm 1,0,3,2
    x = min(x, dpp<0x4E>(~0u, x));                                 // quad_perm 2,3,0,1
    x = min(x, dpp<0x141>(~0u, x));                                // row_half_mirror
    x = min(x, dpp<0x140>(~0u, x));                                // row_mirror
    if constexpr (LPL == 32) {
        const auto r = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        x = min(r[0], r[1]);
    }
    if constexpr (LPL == 64) {
        x = min(x, dpp<0x142>(x, x));                              // row_bcast:15
        x = min(x, dpp<0x143>(x, x));                              // row_bcast:31
        x = (uint32_t)__builtin_amdgcn_readlane((int)x, 63);
    }
    return x;
}

template <int N, class F>
__device__ __forceinline__ void unrolled(F&& f) {
    if constexpr (N > 0) {
        unrolled<N - 1>(f);
        f(std::integral_constant<int, N - 1>{});
    }
}

// One lane's share of a line: 2 R disparities from d0.
template <int LPL, int R>
struct Line {
    // costs above the last minimum: disparities d0 + r and d0 + R + r share a
    // register, so that a neighbour's are another register but at the ends
    uint32_t L[R];
    uint32_t first, last;           // all ones in the line's first / last lane
    uint32_t past;                  // kPast where the lane lies past D
    int d0;

    __device__ __forceinline__ void init(int lane, int D) {
        const int l = lane & (LPL - 1);
        first = l == 0 ? ~0u : 0u;
        last = l == LPL - 1 ? ~0u : 0u;
        d0 = l * 2 * R;
        past = d0 >= D ? kPast : 0u;
#pragma unroll
        for (int r = 0; r < R; ++r) L[r] = 0u;        // then the first step's t is its C
    }

    // Hamming costs of the left word against the lane's right words at
    // column x (INSIDE: no disparity of the wave leaves the image)
    template <bool INSIDE>
    __device__ __forceinline__ void cost(uint64_t left, const uint64_t (&w)[2 * R], int x,
                                         uint32_t (&C)[R]) const {
        const uint32_t l0 = (uint32_t)left, l1 = (uint32_t)(left >> 32);
        uint32_t c[2 * R];
#pragma unroll
        for (int i = 0; i < 2 * R; ++i) {
            c[i] = bit_count(l1 ^ (uint32_t)(w[i] >> 32), bit_count(l0 ^ (uint32_t)w[i], past));
            if (!INSIDE) c[i] = x >= d0 + i ? c[i] : kCostOut + past;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) C[r] = c[r] | (c[R + r] << 16);
    }

    // one step: t becomes the path costs
    __device__ __forceinline__ void step(const uint32_t (&C)[R], uint32_t P1, uint32_t P2,
                                         uint32_t (&t)[R]) {
        const uint32_t B = from_below<LPL>(L[R - 1], first);
        const uint32_t A = from_above<LPL>(L[0], last);
        uint32_t m;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t dn = r > 0 ? L[r - 1] : __builtin_amdgcn_alignbit(L[R - 1], B, 16);
            const uint32_t up = r + 1 < R ? L[r + 1] : __builtin_amdgcn_alignbit(A, L[0], 16);
            const uint32_t n = pk_add(pk_min(dn, up), P1);
            t[r] = pk_add(pk_min3(n, L[r], P2), C[r]);
        }
        if constexpr (R == 4) m = pk_min(pk_min3(t[0], t[1], t[2]), t[3]);
        else m = R == 2 ? pk_min(t[0], t[R - 1]) : t[0];
        // both halves the lane's minimum: then whole words compare alike
        m = pk_min(m, __builtin_amdgcn_alignbit(m, m, 16));
        const uint32_t M = line_min<LPL>(m);
#pragma unroll
        for (int r = 0; r < R; ++r) L[r] = pk_sub(t[r], M);
    }
};

// A lane's offset within a line or a group of columns is below kRange (8192
// columns of 256 disparities, four lines); kNowhere is past it.
constexpr uint32_t kRange = 1u << 24, kNowhere = 1u << 31;

// The lane's 2 R bytes of path costs, in the order of packed_place().
template <int R>
struct Bytes {
    static constexpr int kWords = R > 1 ? R / 2 : 1;
    uint32_t b[kWords];
    __device__ __forceinline__ void pack(const uint32_t (&t)[R]) {
        if constexpr (R == 1) b[0] = __builtin_amdgcn_perm(0u, t[0], 0x0c0c0200u);
        else
#pragma unroll
            for (int i = 0; i < kWords; ++i) b[i] = t[2 * i] | (t[2 * i + 1] << 8);
    }
    // to base + off, or nowhere past kRange: a buffer's range check instead of
    // a branch, so that steps stay one block that the compiler can interleave
    __device__ __forceinline__ void store(uint8_t* base, uint32_t off) const {
        const auto buf = __builtin_amdgcn_make_buffer_rsrc(base, 0, (int)kRange, 0x00027000);
        if constexpr (R == 1)
            __builtin_amdgcn_raw_buffer_store_b16((uint16_t)b[0], buf, (int)off, 0, 0);
        else if constexpr (R == 2)
            __builtin_amdgcn_raw_buffer_store_b32(b[0], buf, (int)off, 0, 0);
        else {
            typedef uint32_t pair __attribute__((ext_vector_type(2)));
            __builtin_amdgcn_raw_buffer_store_b64(pair{b[0], b[1]}, buf, (int)off, 0, 0);
        }
    }
    __device__ __forceinline__ void load(const uint8_t* p) {
        if constexpr (R == 1) b[0] = *reinterpret_cast<const uint16_t*>(p);
        else if constexpr (R == 2) b[0] = *reinterpret_cast<const uint32_t*>(p);
        else {
            typedef uint32_t pair __attribute__((ext_vector_type(2), aligned(4)));
            const pair v = *reinterpret_cast<const pair*>(p);
            b[0] = v[0];
            b[1] = v[1];
        }
    }
    // disparities d0 + r and d0 + R + r, 16 bits each
    __device__ __forceinline__ uint32_t half(int r) const {
        if constexpr (R == 1) return __builtin_amdgcn_perm(0u, b[0], 0x0c010c00u);
        return (r & 1) ? __builtin_amdgcn_perm(0u, b[r / 2], 0x0c030c01u)
                       : __builtin_amdgcn_perm(0u, b[r / 2], 0x0c020c00u);
    }
};

// Keeps a uniform offset in scalar registers, apart from the lane's.
__device__ __forceinline__ size_t uniform(size_t x) {
    return ((size_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(x >> 32)) << 32) |
           (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)x);
}

__device__ __forceinline__ int xcd_contiguous(int b, int n) {
    const int x = b & 7, j = b >> 3, q = n >> 3, r = n & 7;
    return x * q + min(x, r) + j;
}

__device__ __forceinline__ void lds_barrier() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0xc07f);               // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

struct PackedArgs {
    const uint64_t* cl;
    const uint64_t* cr;
    uint8_t* L;                     // planes: down, up, leftwards, rightwards
    size_t plane;                   // bytes of one
    float* disp;
    int W, H, D, P1, P2, frames;
};

// Column lines: G waves take G 64/LPL neighbouring columns and share the
// census words of kRows rows at a time through LDS.  Right words k and k + 2 R
// lie next to each other there: lane l reads the words 2 R l away from lane
// 0's, so a read takes 16 words in a row and no bank twice.
constexpr int kRows = 4;
template <int LPL, int R, int G>
struct ColumnStage {
    static constexpr int kLines = G * (64 / LPL), kRight = 2 * R * LPL + kLines - 1;
    static constexpr int kStride = ((kRight + 2 * R - 1) / (2 * R)) | 1;
    static constexpr int kWords = 2 * R * kStride + kLines;      // of a row, left ones last
    static constexpr int kLoads = (kRows * (kRight + kLines) + 64 * G - 1) / (64 * G);
    uint64_t w[2][kRows * kWords + 1];
    __device__ static int at(int k) { return (k % (2 * R)) * kStride + k / (2 * R); }
};

template <int LPL, int R, int G, bool UP>
__device__ __forceinline__ void column_pass(const PackedArgs& a, ColumnStage<LPL, R, G>& stage,
                                            const int block, uint8_t* plane) {
    using CS = ColumnStage<LPL, R, G>;
    constexpr int Dpad = 2 * R * LPL, LPW = 64 / LPL, kPer = CS::kRight + CS::kLines;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int W = a.W, H = a.H, D = a.D;
    const int groups = (W + CS::kLines - 1) / CS::kLines;
    const int f = block / groups, x0 = (block - f * groups) * CS::kLines;
    const int li = wave * LPW + lane / LPL;           // the line within the group
    const int x = x0 + li;                            // past the last column: not stored
    const size_t fo = (size_t)f * W * H;
    const uint64_t* __restrict__ cl = a.cl + fo;
    const uint64_t* __restrict__ cr = a.cr + fo;
    Line<LPL, R> ln;
    ln.init(lane, D);
    const size_t row = (size_t)W * D;
    // uniform address and the lane's offset from it
    uint8_t* out = plane + (fo + x0) * (size_t)D + (UP ? (size_t)(H - 1) * row : 0);
    const uint32_t off = ln.d0 < D && x < W ? (uint32_t)(li * D + ln.d0) : kNowhere;
    const uint32_t P1 = (uint32_t)a.P1 * 0x10001u, P2 = (uint32_t)a.P2 * 0x10001u;

    // a thread's words: row, source column and place of each
    uint64_t pre[CS::kLoads];
    auto stage_load = [&](int s0) {
#pragma unroll
        for (int k = 0; k < CS::kLoads; ++k) {
            const int idx = min((int)threadIdx.x + k * 64 * G, kRows * kPer - 1);
            const int r = idx / kPer, j = idx - r * kPer;
            const int s = min(s0 + r, H - 1);
            const size_t ro = (size_t)(UP ? H - 1 - s : s) * W;
            pre[k] = j < CS::kRight ? cr[ro + min(max(x0 - Dpad + 1 + j, 0), W - 1)]
                                    : cl[ro + min(x0 + j - CS::kRight, W - 1)];
        }
    };
    auto stage_store = [&](int buf) {
#pragma unroll
        for (int k = 0; k < CS::kLoads; ++k) {
            const int i = (int)threadIdx.x + k * 64 * G;
            const int idx = min(i, kRows * kPer - 1);
            const int r = idx / kPer, j = idx - r * kPer;
            const int at = r * CS::kWords +
                           (j < CS::kRight ? CS::at(j) : 2 * R * CS::kStride + j - CS::kRight);
            stage.w[buf][i < kRows * kPer ? at : kRows * CS::kWords] = pre[k];
        }
    };
    stage_load(0);
    stage_store(0);
    lds_barrier();
    stage_load(kRows);
    int at[2 * R];
#pragma unroll
    for (int i = 0; i < 2 * R; ++i) at[i] = CS::at(li + Dpad - 1 - ln.d0 - i);
    // volatile: one read each, at a constant from the lane's address (pairs of
    // reads reach too few words for that, and would be sums of the vector ALU)
    typedef volatile __attribute__((address_space(3))) uint64_t* lds_words;
    const lds_words words = (lds_words)&stage.w[0][0];
    auto rows = [&](auto INSIDE, auto BUF, int s0) {
        constexpr int base = decltype(BUF)::value * (kRows * CS::kWords + 1);
#pragma unroll
        for (int u = 0; u < kRows; ++u) {
            uint64_t w[2 * R];
#pragma unroll
            for (int i = 0; i < 2 * R; ++i) w[i] = words[base + u * CS::kWords + at[i]];
            const uint64_t lw = words[base + u * CS::kWords + 2 * R * CS::kStride + li];
            uint32_t C[R], t[R];
            ln.template cost<decltype(INSIDE)::value>(lw, w, x, C);
            ln.step(C, P1, P2, t);
            Bytes<R> b;
            b.pack(t);
            b.store(out, decltype(INSIDE)::value || s0 + u < H ? off : kNowhere);
            out = UP ? out - row : out + row;
        }
    };
    // uniform over the workgroup: every disparity of every line inside
    const bool inside = x0 >= Dpad - 1;
    int s0 = 0;
    auto turn = [&](auto INSIDE, auto BUF) {
        constexpr int other = 1 - decltype(BUF)::value;
        rows(INSIDE, BUF, s0);
        stage_store(other);
        lds_barrier();
        stage_load(s0 + 2 * kRows);
        s0 += kRows;
    };
    using Even = std::integral_constant<int, 0>;
    using Odd = std::integral_constant<int, 1>;
    if (inside)
        while (s0 + 2 * kRows <= H) {
            turn(std::true_type{}, Even{});
            turn(std::true_type{}, Odd{});
        }
    while (s0 < H) {
        turn(std::false_type{}, Even{});
        if (s0 < H) turn(std::false_type{}, Odd{});
    }
}

// The words of a row line.  The right-view words of its disparities are the
// last step's moved by one disparity, so a step brings one word; lane l of
// each 16 loads the left and the entering word of step 16 k + l, and a step
// takes them from there (row_word), 8 steps to a turn.
constexpr int kTurn = 8;
template <int LPL, int R, bool RIGHT>
struct RowWords {
    const uint64_t* __restrict__ cl;
    const uint64_t* __restrict__ cr;
    int W, l16;
    uint64_t w[2 * R], left, enter, next_left, next_enter;

    __device__ __forceinline__ void load(int s0) {
        constexpr int Dpad = 2 * R * LPL;
        const int s = min(s0 + l16, W - 1);
        next_left = cl[RIGHT ? s : W - 1 - s];
        // of the step after: disparity 0's, or the window's last one
        next_enter = cr[RIGHT ? min(s + 1, W - 1) : max(W - 2 - s - (Dpad - 1), 0)];
    }
    __device__ __forceinline__ void init(const PackedArgs& a, size_t ro, int lane, int d0) {
        cl = a.cl + ro;
        cr = a.cr + ro;
        W = a.W;
        l16 = lane & 15;
#pragma unroll
        for (int i = 0; i < 2 * R; ++i) w[i] = cr[max((RIGHT ? 0 : W - 1) - (d0 + i), 0)];
        load(0);
    }
    // start of kTurn steps
    __device__ __forceinline__ void turn(int s0) {
        if ((s0 & 15) == 0) {
            left = next_left;
            enter = next_enter;
            load(s0 + 16);
        } else {
            left = upper(left);
            enter = upper(enter);
        }
    }
    __device__ static uint64_t upper(uint64_t x) {    // row_shl:8
        return ((uint64_t)dpp<0x108>(0u, (uint32_t)(x >> 32)) << 32) | dpp<0x108>(0u, (uint32_t)x);
    }
    template <int U>
    __device__ __forceinline__ void slide(const Line<LPL, R>& ln) {
        constexpr int C = LPL == 16 ? (RIGHT ? 0x111 : 0x101) : (RIGHT ? 0x138 : 0x130);
        const uint64_t e = row_word<U>(enter);
        const uint64_t v = RIGHT ? w[2 * R - 1] : w[0];
        uint32_t lo = dpp<C>((uint32_t)e, (uint32_t)v);
        uint32_t hi = dpp<C>((uint32_t)(e >> 32), (uint32_t)(v >> 32));
        if constexpr (LPL == 32) {                    // the inner line's edge lane
            const bool edge = (RIGHT ? ln.first : ln.last) != 0u;
            lo = edge ? (uint32_t)e : lo;
            hi = edge ? (uint32_t)(e >> 32) : hi;
        }
        const uint64_t in = ((uint64_t)hi << 32) | lo;
        if constexpr (RIGHT) {
#pragma unroll
            for (int i = 2 * R - 1; i > 0; --i) w[i] = w[i - 1];
            w[0] = in;
        } else {
#pragma unroll
            for (int i = 0; i < 2 * R - 1; ++i) w[i] = w[i + 1];
            w[2 * R - 1] = in;
        }
    }
};

// Right-to-left rows where lines are many: block of G waves, 64 / LPL rows each.
template <int LPL, int R, int G>
__device__ __forceinline__ void row_pass(const PackedArgs& a, const int block, uint8_t* plane) {
    constexpr int Dpad = 2 * R * LPL, LPW = 64 / LPL;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int W = a.W, D = a.D, lines = a.H * a.frames;
    const int first = (block * G + wave) * LPW;
    if (first >= lines) return;
    const int line = min(first + lane / LPL, lines - 1);
    const size_t ro = (size_t)line * W;
    Line<LPL, R> ln;
    ln.init(lane, D);
    // uniform address and the lane's offset from it
    uint8_t* out = plane + ((size_t)first * W + W - 1) * (size_t)D;
    const uint32_t off = ln.d0 < D && first + lane / LPL < lines
                             ? (uint32_t)((line - first) * W * D + ln.d0) : kNowhere;
    const uint32_t P1 = (uint32_t)a.P1 * 0x10001u, P2 = (uint32_t)a.P2 * 0x10001u;
    RowWords<LPL, R, false> rw;
    rw.init(a, ro, lane, ln.d0);
    auto steps = [&](auto INSIDE, int s0) {
        unrolled<kTurn>([&](auto U) {
            constexpr int u = decltype(U)::value;
            const int s = s0 + u;
            uint32_t C[R], t[R];
            ln.template cost<decltype(INSIDE)::value>(row_word<u>(rw.left), rw.w,
                                                      W - 1 - s, C);
            ln.step(C, P1, P2, t);
            Bytes<R> b;
            b.pack(t);
            b.store(out, decltype(INSIDE)::value || s < W ? off : kNowhere);
            out -= D;
            rw.template slide<u>(ln);
        });
    };
    // checked steps near the image's left edge and past its last full turn, as
    // loops of their own: as the sides of a branch in one loop, each side's
    // state would live through the other's
    int s0 = 0;
    for (; W - kTurn - s0 >= Dpad - 1; s0 += kTurn) {
        rw.turn(s0);
        steps(std::true_type{}, s0);
    }
    for (; s0 < W; s0 += kTurn) {
        rw.turn(s0);
        steps(std::false_type{}, s0);
    }
}

// Rows where lines are few: a pair of waves per row, one that forms the Hamming
// costs kTurn steps ahead (double-buffered in LDS), one that runs the
// recurrence over them, whose chain bounds the call.  Against a wave that does
// both, a row spread over all its 64 lanes (two disparities each): 1024x440 and
// 128 disparities 218 -> 190 us at one pair, 699 -> 616 at four; 641x241 and 64
// 115 -> 85 at one.  (Columns in such pairs as well: 214 and 640.)
template <int R, int G>
struct PairStage {
    uint32_t c[G / 2][2][kTurn * R * 64];
};

template <int LPL, int R, int G, bool RIGHT>
__device__ __forceinline__ void row_pair_pass(const PackedArgs& a, PairStage<R, G>& stage,
                                              const int block, uint8_t* plane) {
    constexpr int Dpad = 2 * R * LPL, LPW = 64 / LPL;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int W = a.W, D = a.D, lines = a.H * a.frames;
    // the roles change places from block to block, so that neighbours on a
    // compute unit don't put their chains on the same SIMDs
    const int role = ((wave & 1) ^ (block & 1)), pair = wave >> 1;
    const int first = min((block * (G / 2) + pair) * LPW, lines - 1);
    const int line = min(first + lane / LPL, lines - 1);
    const bool real = (block * (G / 2) + pair) * LPW + lane / LPL < lines;
    const size_t ro = (size_t)line * W;
    Line<LPL, R> ln;
    ln.init(lane, D);
    const int turns = (W + kTurn - 1) / kTurn;
    uint32_t* const mine = &stage.c[pair][0][lane];
    if (role == 0) {
        RowWords<LPL, R, RIGHT> rw;
        rw.init(a, ro, lane, ln.d0);
        auto turn = [&](auto INSIDE, int t) {
            const int s0 = t * kTurn;
            rw.turn(s0);
            uint32_t* const to = mine + (t & 1) * kTurn * R * 64;
            unrolled<kTurn>([&](auto U) {
                constexpr int u = decltype(U)::value;
                uint32_t C[R];
                const int s = s0 + u;
                ln.template cost<decltype(INSIDE)::value>(row_word<u>(rw.left), rw.w,
                                                          RIGHT ? s : W - 1 - s, C);
#pragma unroll
                for (int r = 0; r < R; ++r) to[(u * R + r) * 64] = C[r];
                rw.template slide<u>(ln);
            });
            lds_barrier();
        };
        int t = 0;
        if (RIGHT)
            for (; t < turns && t * kTurn < Dpad - 1; ++t) turn(std::false_type{}, t);
        for (; RIGHT ? t < turns : (t < turns && W - kTurn - t * kTurn >= Dpad - 1); ++t)
            turn(std::true_type{}, t);
        for (; t < turns; ++t) turn(std::false_type{}, t);
    } else {
        // uniform address and the lane's offset from it
        uint8_t* out = plane + ((size_t)first * W + (RIGHT ? 0 : W - 1)) * (size_t)D;
        const uint32_t off =
            ln.d0 < D && real ? (uint32_t)((line - first) * W * D + ln.d0) : kNowhere;
        const uint32_t P1 = (uint32_t)a.P1 * 0x10001u, P2 = (uint32_t)a.P2 * 0x10001u;
        auto turn = [&](auto FULL, int t) {
            lds_barrier();
            const uint32_t* const from = mine + (t & 1) * kTurn * R * 64;
            uint32_t C[kTurn][R];
#pragma unroll
            for (int u = 0; u < kTurn; ++u)
#pragma unroll
                for (int r = 0; r < R; ++r) C[u][r] = from[(u * R + r) * 64];
#pragma unroll
            for (int u = 0; u < kTurn; ++u) {
                uint32_t c[R];
                ln.step(C[u], P1, P2, c);
                Bytes<R> b;
                b.pack(c);
                b.store(out, decltype(FULL)::value || t * kTurn + u < W ? off : kNowhere);
                out = RIGHT ? out + D : out - D;
            }
        };
        for (int t = 0; t < turns - 1; ++t) turn(std::true_type{}, t);
        turn(std::false_type{}, turns - 1);
    }
}

// The directions whose costs go to memory, as ranges of blocks; the rows'
// lines are the longest, so their blocks go first.
template <int LPL, int R, int G, bool FOUR>
__global__ __launch_bounds__(64 * G) void paths_kernel(PackedArgs a, int row_blocks, int col_blocks) {
    using Columns = ColumnStage<LPL, R, G>;
    using Rows = PairStage<R, G>;
    constexpr size_t kShared = !FOUR || sizeof(Columns) > sizeof(Rows) ? sizeof(Columns) : sizeof(Rows);
    __shared__ __attribute__((aligned(16))) char shared[kShared];
    Columns& stage = *reinterpret_cast<Columns*>(shared);
    int b = (int)blockIdx.x;
    if constexpr (FOUR) {
        Rows& pairs = *reinterpret_cast<Rows*>(shared);
        if (b < 2 * row_blocks) {
            // a row's two directions next to each other
            const int r = xcd_contiguous(b, 2 * row_blocks);
            if (r & 1)
                row_pair_pass<LPL, R, G, true>(a, pairs, r >> 1, a.L + 3 * a.plane);
            else
                row_pair_pass<LPL, R, G, false>(a, pairs, r >> 1, a.L + 2 * a.plane);
            return;
        }
        b -= 2 * row_blocks;
    } else {
        if (b < row_blocks) {
            row_pass<LPL, R, G>(a, xcd_contiguous(b, row_blocks), a.L + 2 * a.plane);
            return;
        }
        b -= row_blocks;
    }
    if (b < col_blocks)
        column_pass<LPL, R, G, false>(a, stage, xcd_contiguous(b, col_blocks), a.L);
    else
        column_pass<LPL, R, G, true>(a, stage, xcd_contiguous(b - col_blocks, col_blocks),
                                         a.L + a.plane);
}

// A line's selection keys, sum << 16 | d, of one column, the left view's
// minimum over the line, and the right view's: its minimum of column x' = x - d
// moves along the disparities with x, so that it needs no shared memory until
// it is complete at the last one.
template <int LPL, int R>
struct Selection {
    uint32_t acc[2 * R];
    uint32_t skip;                  // all ones past D: no key

    __device__ __forceinline__ void init(const Line<LPL, R>& ln, int D) {
        skip = ln.d0 >= D ? ~0u : 0u;
#pragma unroll
        for (int i = 0; i < 2 * R; ++i) acc[i] = ~0u;
    }
    // The minima so far: two steps' become one three-way minimum, later ones are
    // not put off (their keys would wait in registers).
    __device__ __forceinline__ void settle() {
#pragma unroll
        for (int i = 0; i < 2 * R; ++i) asm volatile("" : "+v"(acc[i]));
    }
    __device__ __forceinline__ uint32_t step(const uint32_t (&s)[R], const Line<LPL, R>& ln,
                                             uint32_t none) {
        uint32_t key[2 * R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            key[r] = (s[r] << 16) | (uint32_t)(ln.d0 + r) | none;
            key[R + r] = (s[r] & 0xffff0000u) | (uint32_t)(ln.d0 + R + r) | none;
        }
        uint32_t k = key[0];
#pragma unroll
        for (int i = 1; i < 2 * R; ++i) k = min(k, key[i]);
        const uint32_t in = from_below<LPL>(acc[2 * R - 1], ln.first);
#pragma unroll
        for (int i = 2 * R - 1; i > 0; --i) acc[i] = min(acc[i - 1], key[i]);
        acc[0] = min(in, key[0]);
        return line_min<LPL>(k | skip);
    }
};

constexpr int kAhead = 4;           // columns whose path costs are on their way

// Left to right, selection and check: one wave per block, 64 / LPL rows.
template <int LPL, int R>
__global__ __launch_bounds__(64, 4) void final_path_kernel(PackedArgs a) {
    constexpr int Dpad = 2 * R * LPL, LPW = 64 / LPL;
    extern __shared__ uint8_t sel[];                  // per line: d_L [Wp], d_R [Wp + 8]
    const int lane = threadIdx.x & 63;
    const int W = a.W, D = a.D, lines = a.H * a.frames;
    const int Wp = (W + 7) & ~3;
    const int first_line = xcd_contiguous((int)blockIdx.x, (int)gridDim.x) * LPW;
    const int line = min(first_line + lane / LPL, lines - 1);
    const size_t ro = (size_t)line * W;
    Line<LPL, R> ln;
    ln.init(lane, D);
    uint8_t* const dL = sel + (lane / LPL) * (2 * Wp + 8);
    uint8_t* const dR = dL + Wp;                      // column x' at x' + 4
    const uint32_t P1 = (uint32_t)a.P1 * 0x10001u, P2 = (uint32_t)a.P2 * 0x10001u;
    const bool leader = ln.first != 0u;               // writes d_L
    const bool drain = ln.d0 == D - 2 * R;            // holds disparity D - 1: writes d_R
    // planes: a uniform address and the lane's offset from it (lanes past D
    // repeat the last costs)
    const uint8_t* const q0 = a.L + (size_t)first_line * W * D;
    const uint8_t* const q1 = q0 + a.plane;
    const uint8_t* const q2 = q1 + a.plane;
    const uint32_t off = (uint32_t)((line - first_line) * W * D + min(ln.d0, D - 2 * R));
    RowWords<LPL, R, true> rw;
    rw.init(a, ro, lane, ln.d0);
    Bytes<R> b0[kAhead], b1[kAhead], b2[kAhead];
    auto load = [&](int u, int x) {
        const size_t o = uniform((size_t)min(x, W - 1) * D);
        b0[u].load(q0 + o + off);
        b1[u].load(q1 + o + off);
        b2[u].load(q2 + o + off);
    };
#pragma unroll
    for (int u = 0; u < kAhead; ++u) load(u, u);
    Selection<LPL, R> pick;
    pick.init(ln, D);
    auto steps = [&](auto INSIDE, int x0) {
        uint32_t l4 = 0, r4 = 0;                      // four columns' bytes
        unrolled<kTurn>([&](auto U) {
            constexpr int u = decltype(U)::value, v = u % kAhead;
            const int x = x0 + u;
            uint32_t C[R], s[R];
            ln.template cost<decltype(INSIDE)::value>(row_word<u>(rw.left), rw.w, x, C);
            ln.step(C, P1, P2, s);
            rw.template slide<u>(ln);
#pragma unroll
            for (int r = 0; r < R; ++r)
                s[r] = pk_add(pk_add(s[r], b0[v].half(r)), pk_add(b1[v].half(r), b2[v].half(r)));
            load(v, x + kAhead);
            const uint32_t k = pick.step(s, ln, decltype(INSIDE)::value || x < W ? 0u : ~0u);
            l4 |= (k & 0xffu) << (8 * (u & 3));
            r4 |= (pick.acc[2 * R - 1] & 0xffu) << (8 * (u & 3));
            if constexpr ((u & 3) == 3) {
                if (leader && (decltype(INSIDE)::value || x - 3 < W))
                    *reinterpret_cast<uint32_t*>(dL + x - 3) = l4;
                // columns x - D - 2 .. x - D + 1, at + 4: those outside the image land
                // in front or behind
                if (drain && (decltype(INSIDE)::value || (x >= D - 1 && x - D < W + 3))) {
                    uint8_t* const p = dR + (x - D + 2);
                    p[0] = (uint8_t)r4;
                    p[1] = (uint8_t)(r4 >> 8);
                    p[2] = (uint8_t)(r4 >> 16);
                    p[3] = (uint8_t)(r4 >> 24);
                }
                l4 = r4 = 0;
            }
            if constexpr (u & 1) pick.settle();
        });
    };
    int x0 = 0;
    for (; x0 < min(W, Dpad - 1); x0 += kTurn) {
        rw.turn(x0);
        steps(std::false_type{}, x0);
    }
    for (; x0 + kTurn <= W; x0 += kTurn) {
        rw.turn(x0);
        steps(std::true_type{}, x0);
    }
    for (; x0 < W; x0 += kTurn) {
        rw.turn(x0);
        steps(std::false_type{}, x0);
    }
    // the last columns' minima are still on their way
#pragma unroll
    for (int i = 0; i < 2 * R; ++i) {
        const int x = x0 - 1 - (ln.d0 + i);
        if (ln.d0 < D && x >= 0 && x < W) dR[x + 4] = (uint8_t)pick.acc[i];
    }
    __syncthreads();
    for (int l = 0; l < LPW; ++l) {
        if (first_line + l >= lines) break;
        const uint8_t* const el = sel + l * (2 * Wp + 8);
        float* const o = a.disp + (size_t)(first_line + l) * W;
        for (int x = lane; x < W; x += 64) {
            const int d = el[x];
            float v = -1.0f;
            if (x - d >= 0 && abs(d - (int)el[Wp + x - d + 4]) <= 1) v = (float)d;
            o[x] = v;
        }
    }
}

// Selection and check where all four directions are in memory: a workgroup per
// row, its kSelectWaves * 64 / LPL lines a segment of the columns each.
constexpr int kSelectWaves = 8;
template <int LPL, int R>
__global__ __launch_bounds__(64 * kSelectWaves) void select_kernel(PackedArgs a) {
    constexpr int LPW = 64 / LPL, kSegments = kSelectWaves * LPW, kThreads = 64 * kSelectWaves;
    extern __shared__ uint32_t rkey[];                // right view's keys [W], then d_L [W] bytes
    const int W = a.W, D = a.D;
    uint8_t* const dL = reinterpret_cast<uint8_t*>(rkey + W);
    const int row = xcd_contiguous((int)blockIdx.x, (int)gridDim.x);
    for (int x = (int)threadIdx.x; x < W; x += kThreads) rkey[x] = ~0u;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int seg = (W + kSegments - 1) / kSegments;
    Line<LPL, R> ln;
    ln.init(lane, D);
    const int sub = lane / LPL, x0 = (wave * LPW + sub) * seg;
    const uint8_t* q[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) q[r] = a.L + (size_t)r * a.plane + (size_t)row * W * D;
    const uint32_t d = (uint32_t)min(ln.d0, D - 2 * R);
    Bytes<R> b[kAhead][4];
    auto load = [&](int u, int s) {
        const uint32_t off = (uint32_t)(min(x0 + min(s, seg - 1), W - 1) * D) + d;
#pragma unroll
        for (int r = 0; r < 4; ++r) b[u][r].load(q[r] + off);
    };
#pragma unroll
    for (int u = 0; u < kAhead; ++u) load(u, u);
    Selection<LPL, R> pick;
    pick.init(ln, D);
    const bool leader = ln.first != 0u, drain = ln.d0 == D - 2 * R;
    __syncthreads();
    int x = x0;
    for (int s0 = 0; s0 < seg; s0 += kAhead) {
#pragma unroll
        for (int u = 0; u < kAhead; ++u, ++x) {
            if (s0 + u < seg) {                       // uniform
                uint32_t s[R];
#pragma unroll
                for (int r = 0; r < R; ++r)
                    s[r] = pk_add(pk_add(b[u][0].half(r), b[u][1].half(r)),
                                  pk_add(b[u][2].half(r), b[u][3].half(r)));
                load(u, s0 + u + kAhead);
                const uint32_t k = pick.step(s, ln, x < W ? 0u : ~0u);
                if (leader && x < W) dL[x] = (uint8_t)k;
                const int c = x - D + 1;
                if (drain && c >= 0 && c < W) atomicMin(&rkey[c], pick.acc[2 * R - 1]);
            }
        }
    }
    x = x0 + seg - 1;
    // the last columns' minima are still on their way, and the next segments add theirs
#pragma unroll
    for (int i = 0; i < 2 * R; ++i) {
        const int c = x - (ln.d0 + i);
        if (ln.d0 < D && c >= 0 && c < W) atomicMin(&rkey[c], pick.acc[i]);
    }
    __syncthreads();
    float* const o = a.disp + (size_t)row * W;
    for (int i = (int)threadIdx.x; i < W; i += kThreads) {
        const int e = dL[i];
        float v = -1.0f;
        if (i - e >= 0 && abs(e - (int)(rkey[i - e] & 0xffu)) <= 1) v = (float)e;
        o[i] = v;
    }
}

// Batches: lines of as many disparities per lane as there are, three directions
// in memory and the last one fused with the selection.
template <int LPL, int R, int G>
hipError_t launch_many(const PackedArgs& a, hipStream_t st) {
    constexpr int LPW = 64 / LPL;
    const int col = a.frames * ((a.W + G * LPW - 1) / (G * LPW));
    const int lines = a.H * a.frames;
    const int row = (lines + G * LPW - 1) / (G * LPW);
    hipLaunchKernelGGL((paths_kernel<LPL, R, G, false>), dim3((unsigned)(row + 2 * col)),
                       dim3(64 * G), 0, st, a, row, col);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const size_t lds = (size_t)LPW * (2 * (size_t)((a.W + 7) & ~3) + 8);
    hipLaunchKernelGGL((final_path_kernel<LPL, R>), dim3((unsigned)((lines + LPW - 1) / LPW)),
                       dim3(64), lds, st, a);
    return hipGetLastError();
}

// Few lines: a pair of waves per rows, all four directions at once.
template <int LPL, int R>
hipError_t launch_few(const PackedArgs& a, hipStream_t st) {
    constexpr int G = 4, LPW = 64 / LPL;
    const int col = a.frames * ((a.W + G * LPW - 1) / (G * LPW));
    const int lines = a.H * a.frames;
    const int row = (lines + G / 2 * LPW - 1) / (G / 2 * LPW);
    hipLaunchKernelGGL((paths_kernel<LPL, R, G, true>), dim3((unsigned)(2 * (row + col))),
                       dim3(64 * G), 0, st, a, row, col);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((select_kernel<LPL, R>), dim3((unsigned)lines), dim3(64 * kSelectWaves),
                       (size_t)a.W * 5, st, a);
    return hipGetLastError();
}

}  // namespace

bool packed_costs(int P2) { return kCostOut + P2 <= 255; }

// Eight disparities to a lane: lanes then end at D, and four rows of up to 4096
// columns to a wave have their selection state in LDS.
static bool packed_eights(int D, int W) { return D % 8 == 0 && D > 64 && (D > 128 || W <= 4096); }

int packed_place(int D, int W, int d) {
    // a lane's eight: 0 1 4 5, 2 3 6 7
    constexpr int place[8] = {0, 1, 4, 5, 2, 3, 6, 7};
    return packed_eights(D, W) ? (d & ~7) | place[d & 7] : d;
}

// Few lines are all four directions side by side: while a compute unit has at
// most 17 rows of 64 disparities, 14 of 128 or 8 of 256.  On 256 of them, us with
// few / many lines' kernels: 640x240 and 32 disparities 289 / 347 at 16 pairs,
// 581 / 538 at 32; 641x241 and 64: 469 / 518 at 16, 707 / 600 at 24; 1024x440 and
// 128: 617 / 839 at four, 1,081 / 1,219 at eight, 1,589 / 1,420 at twelve;
// 2048x880 and 256: 1,170 / 1,748 at one, 2,115 / 2,518 at two, 3,163 / 2,913 at
// three.
bool packed_four(int D, int H, int frames, int num_cu) {
    return (int64_t)H * frames <= (int64_t)num_cu * (D <= 64 ? 17 : (D <= 128 ? 14 : 8));
}

hipError_t launch_packed_paths(const uint64_t* cl, const uint64_t* cr, uint8_t* planes,
                               size_t plane, bool four, int W, int H, int frames, int D, int P1,
                               int P2, float* disp, hipStream_t st) {
    const PackedArgs a{cl, cr, planes, plane, disp, W, H, D, P1, P2, frames};
    const bool eights = packed_eights(D, W);
    if (four) {
        if (D <= 32) return launch_few<16, 1>(a, st);
        if (D <= 64) return launch_few<16, 2>(a, st);
        if (D <= 128) return eights ? launch_few<16, 4>(a, st) : launch_few<32, 2>(a, st);
        return eights ? launch_few<32, 4>(a, st) : launch_few<64, 2>(a, st);
    }
    // four rows' selection state within 64 KB of LDS: fewer rows to a wave past
    // 4096 columns
    if (D <= 32 && W <= 4096) return launch_many<16, 1, 8>(a, st);
    if (D <= 64 && W <= 4096) return launch_many<16, 2, 8>(a, st);
    if (D <= 128) return eights ? launch_many<16, 4, 8>(a, st) : launch_many<32, 2, 8>(a, st);
    return eights ? launch_many<32, 4, 8>(a, st) : launch_many<64, 2, 8>(a, st);
}

}  // namespace stx::sgm
