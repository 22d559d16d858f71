// chain_frame.hip -- launches with few columns as one kernel: each column is
// reduced, tabulated, solved and backtracked by one workgroup of up to 16 waves
// (Sec. 4.1-4.4 in chain.h's form).
//
// The small prefix tables go straight to the LDS arrays the chain reads, the
// object prefix table to memory (a column's own place, read back through the
// compute unit's caches), its entries at block boundaries to LDS for the
// bounds.  Against three kernels (reduction, tables, recurrence) this takes
// out two launches, their gaps and the tables' way to and from memory.
#include <algorithm>
#include <climits>

#include "arena.h"
#include "chain.h"
#include "chain_frame.h"

namespace stx::persist {

namespace {

enum { kFrame = 0, kBatch = 1, kArena = 2, kArenaRest = 3 };

// Device header of a frame whose tables share a workspace (kArena): the next
// column, floats handed out, the columns left over and the next of those.
struct ArenaHead {
    unsigned int next, used4, nrest, next_rest;
};

struct ChainArgs {
    JobDesc job;                 // kFrame, kArena, kArenaRest
    ChainExports ex;             // kFrame
    const JobDesc* jobs;         // kBatch
    const int2* tasks;
    int ntasks;
    unsigned int* counter;
    float* po;
    long long stride;            // floats between tables (kFrame, kBatch, kArenaRest)
    ArenaHead* head;             // kArena, kArenaRest
    int* rest;
    unsigned int room4;          // kArena: 16-byte units of table space
};

// The kernel's arguments and the jobs are read where they are used, through
// the scalar cache: kept over a column (or over the loop of columns) they fill
// the scalar registers, whose overflow then fills the vector registers, inside
// the recurrence's loops (the batch form spilled 31 and the workspace form 81
// vector registers, now 9 and 7: 64 uneven frames 4,170 -> 3,644 us, 1024x437
// at half pixels in a workspace 96 -> 73).
template <class T>
using Const = const __attribute__((address_space(4))) T*;
template <class T>
__device__ __forceinline__ Const<T> in_const(const T* p) {
    return (Const<T>)reinterpret_cast<uintptr_t>(p);
}
// p, with everything read through it so far forgotten
template <class T>
__device__ __forceinline__ Const<T> again(Const<T> p) {
    asm volatile("" : "+s"(p));
    return p;
}
template <class T>
__device__ __forceinline__ T load_const(Const<T> p) {
    static_assert(sizeof(T) % 4 == 0, "whole words");
    struct Words {
        uint32_t w[sizeof(T) / 4];
    } x;
#pragma unroll
    for (int i = 0; i < (int)(sizeof(T) / 4); ++i) x.w[i] = ((Const<uint32_t>)p)[i];
    return __builtin_bit_cast(T, x);
}

// LDS besides the chain's: the overlay of the ring and records holds, until
// the chain starts, the edges (D rows), a staged cost row per wave and the
// column's pixels.
__host__ __device__ constexpr int overlay_bytes(int H, int D, int nw) {
    return D * (H / kBlock / 4 + 1) * 16 + nw * (kMaxDisparity + 4) * 4 + ((H + 7) & ~7) * 2;
}
__host__ __device__ constexpr int ring_rec_bytes(int H) {
    return kRing * kGroup * 64 * 16 + chain_rows(H) * 16;
}
// the chain's arrays after the overlay start higher when the overlay is the
// larger of the two
__host__ __device__ constexpr int lds_bytes(int H, int D, int nw) {
    const int more = overlay_bytes(H, D, nw) - ring_rec_bytes(H);
    return (int)chain_lds_bytes(H) + (more > 0 ? ((more + 15) & ~15) : 0);
}

// ... and the kernels' own variables: four words, and two more, padded, where
// columns are handed out.
constexpr int static_lds(bool frame) { return frame ? 16 : 32; }

// Small prefix table t of a column from its pixels (one wave): entries into a
// component of an LDS float4 array, and to memory when out is given.
__device__ __forceinline__ void small_table(Const<JobDesc> J, const int16_t* qs, const int t,
                                            float* dst, float* out) {
    const int lane = threadIdx.x & 63;
    const int H = J->H, D = J->D;
    const float* const src = t == 0 ? J->ground : (t == 1 ? J->sky : J->object_min);
    if (lane == 0) {
        dst[0] = 0.0f;
        if (out) out[0] = 0.0f;
    }
    float carry = 0.0f;
#pragma unroll 1
    for (int v0 = 0; v0 < H; v0 += 256) {
        float r[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int v = v0 + 4 * lane + i;
            const int x = (v < H) ? (int)qs[v] : -1;
            r[i] = 0.0f;
            if (x >= 0) {
                r[i] = (t == 2) ? (float)(2 * x + 1)
                     : (t == 3) ? 2.0f
                                : src[(t == 0) ? (size_t)(H - 1 - v) * D + x : (size_t)x];
            }
        }
        r[1] += r[0];
        r[2] += r[1];
        r[3] += r[2];
        const float incl = wave_inclusive_scan(r[3]);
        const float e = (incl - r[3]) + carry;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int v = v0 + 4 * lane + i;
            if (v < H) {
                dst[4 * (v + 1)] = r[i] + e;
                if (out) out[v + 1] = r[i] + e;
            }
        }
        carry = readlane_f(incl, 63) + carry;
    }
}

// Object prefix rows of a column, taken in turn by the waves that are free
// (*next, in LDS): as in the staged table kernel, with the entries 32 i into
// the staged edges.  NU: 256-row groups.
template <int NU>
__device__ __forceinline__ void object_rows(Const<JobDesc> J, const int16_t* qs, float* stg,
                                            float* edges, int* next, float* PO, const int fmin,
                                            const int fmax) {
    constexpr int NC = kMaxDisparity / 64;
    const int lane = threadIdx.x & 63;
    const int H = J->H, D = J->D, nch = (D + 63) >> 6, nq4 = 4 * chain_edge_quads(H);
    const uint32_t stride4 = (uint32_t)po_row_floats(H) * 4u;
    const auto otr = make_rsrc(J->object_t, (uint32_t)(D * D) * 4u);
    const auto pow_ = make_rsrc(PO, (uint32_t)(fmax - fmin + 1) * stride4);
    if (lane == 0) stg[D] = 0.0f;
    int qi[NU][4];                               // stage index of each row's cost
#pragma unroll
    for (int u = 0; u < NU; ++u) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int v = 256 * u + 4 * lane + i;
            const int x = (v < H) ? (int)qs[v] : -1;
            qi[u][i] = (x >= 0) ? x : D;
        }
    }
    auto take = [&]() {
        int n = 0;
        if (lane == 0) n = atomicAdd(next, 1);
        return fmin + __builtin_amdgcn_readfirstlane(n);
    };
    float onext[NC];
    auto load_row = [&](int f) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if (c >= nch) break;
            onext[c] = buf_load_b(otr, (uint32_t)(64 * c + lane) * 4u, (uint32_t)(f * D) * 4u);
        }
    };
    int f = take();
    if (f <= fmax) load_row(f);
#pragma unroll 1
    while (f <= fmax) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if (c >= nch) break;
            if (64 * c + lane < D) stg[64 * c + lane] = onext[c];
        }
        const int fn = take();
        if (fn <= fmax) load_row(fn);
        const uint32_t rowoff = (uint32_t)(f - fmin) * stride4;
        float* const ed = edges + (f - fmin) * nq4;
        if (lane == 0) {
            buf_store_b(pow_, 0.0f, 12u, rowoff);
            ed[0] = 0.0f;
        }
        float carry = 0.0f;
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const float o0 = stg[qi[u][0]], o1 = stg[qi[u][1]];
            const float o2 = stg[qi[u][2]], o3 = stg[qi[u][3]];
            const float a1 = o0 + o1, a2 = a1 + o2, a3 = a2 + o3;
            const float incl = wave_inclusive_scan(a3);
            const float e = (incl - a3) + carry;
            const int v = 256 * u + 4 * lane;    // the lane's first row
            if (v < H)
                buf_store_b4(pow_, e + o0, e + a1, e + a2, e + a3, (uint32_t)(v + 4) * 4u, rowoff);
            if ((lane & 7) == 7 && v + 4 <= H) ed[(v + 4) / kBlock] = e + a3;
            carry = readlane_f(incl, 63) + carry;
        }
        f = fn;
    }
}

}  // namespace

template <int MODE>
__global__ __launch_bounds__(64 * kChainWaves)
__attribute__((amdgpu_waves_per_eu(4))) void chain_frame_kernel(const ChainArgs) {
    extern __shared__ __align__(16) char mem[];
    __shared__ int red[4];                       // smallest, largest, any invalid; next object row
    __shared__ int task;
    __shared__ unsigned int place;               // kArena: in 16-byte units
    // the arguments where they lie
    const Const<ChainArgs> a = (Const<ChainArgs>)__builtin_amdgcn_kernarg_segment_ptr();
    const int tid = threadIdx.x, lane = tid & 63, nt = (int)blockDim.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = nt >> 6;
    unsigned int own = 0, own4 = 0;              // kArena: this workgroup's table space,
    bool full = false;                           // and whether it was refused more
#ifdef STX_PHASE_TIMING
    // wave 0 stamps the shader clock at each phase boundary of a batch's column
    const unsigned long long t_entry = __builtin_amdgcn_s_memtime();
    unsigned long long* phases = nullptr;
    unsigned long long t0 = 0, t1 = 0, t2 = 0, t3 = 0, t4 = 0;
    auto phase_add = [&](int slot, unsigned long long v) {
        if (MODE == kBatch && tid == 0 && phases) atomicAdd(phases + slot, v);
    };
#endif
    for (bool once = true; MODE != kFrame || once; once = false) {
        int job = 0, col = (int)blockIdx.x;
        if constexpr (MODE != kFrame) {
            if (tid == 0) {
                const Const<ChainArgs> A = again(a);
                unsigned int* const c = MODE == kBatch ? A->counter
                                      : (MODE == kArena ? &A->head->next : &A->head->next_rest);
                task = (int)atomicAdd(c, 1u);
            }
            __syncthreads();
            const int t = __builtin_amdgcn_readfirstlane(task);
            if constexpr (MODE == kBatch) {
                if (t >= again(a)->ntasks) break;
                const Const<int> tk = in_const(reinterpret_cast<const int*>(again(a)->tasks)) + 2 * t;
                job = tk[0];
                col = tk[1];
            } else if constexpr (MODE == kArena) {
                if (t >= again(a)->job.ncols) break;
                col = t;
            } else {
                const Const<ChainArgs> A = again(a);
                if (t >= __builtin_amdgcn_readfirstlane((int)A->head->nrest)) break;
                col = __builtin_amdgcn_readfirstlane(A->rest[t]);
            }
        }
        const Const<JobDesc> job_at = MODE == kBatch ? in_const(again(a)->jobs) + job : &a->job;
        const int H = job_at->H, D = job_at->D, stride = H + 1;
#ifdef STX_PHASE_TIMING
        phases = job_at->phase;
        t0 = __builtin_amdgcn_s_memtime();
#endif
        ChainLds L = chain_lds(mem, H);
        {   // the overlay may need more room than the ring and the records
            const int more = overlay_bytes(H, D, nw) - ring_rec_bytes(H);
            const int up = more > 0 ? ((more + 15) & ~15) : 0;
            L.bound = reinterpret_cast<float*>(reinterpret_cast<char*>(L.bound) + up);
            L.sum = reinterpret_cast<float4*>(reinterpret_cast<char*>(L.sum) + up);
            L.fl = reinterpret_cast<ChainFlags*>(reinterpret_cast<char*>(L.fl) + up);
        }
        float* const edges = chain_edges(L);
        float* const stage = edges + D * 4 * chain_edge_quads(H);
        int16_t* const qs = reinterpret_cast<int16_t*>(stage + nw * (kMaxDisparity + 4));
        if (tid < 4) red[tid] = tid == 0 ? INT_MAX : (tid == 1 ? -1 : 0);
        chain_clear(L);
        __syncthreads();

        // Sec. 4.1: the column's strips, bottom-up
        int lmin = INT_MAX, lmax = -1;
        bool inv = false;
        const Const<JobDesc> J = again(job_at);
        for (int v = tid; v < H; v += nt) {
            const int x = reduce_any(J->disp + (size_t)(H - 1 - v) * J->W + (size_t)col * J->s, J->s,
                                     J->reduce_mode, D, J->sub);
            qs[v] = (int16_t)x;
            if constexpr (MODE == kFrame) {
                if (a->ex.q) a->ex.q[(size_t)col * H + v] = (int16_t)x;
            }
            if (x >= 0) {
                lmin = min(lmin, x);
                lmax = max(lmax, x);
            } else {
                inv = true;
            }
        }
        lmin = wave_min_i(lmin);
        lmax = wave_max_i(lmax);
        const bool anyinv = __ballot(inv) != 0;
        if (lane == 0) {
            atomicMin(&red[0], lmin);
            atomicMax(&red[1], lmax);
            if (anyinv) atomicOr(&red[2], 1);
        }
        __syncthreads();
#ifdef STX_PHASE_TIMING
        t1 = __builtin_amdgcn_s_memtime();
#endif
        // object means lie in [smallest, largest valid q]; a stixel without
        // valid pixels has mean 0
        int fmin = __builtin_amdgcn_readfirstlane(red[2] ? 0 : red[0]);
        int fmax = __builtin_amdgcn_readfirstlane(red[1]);
        if (fmax < 0) {
            fmin = 0;
            fmax = 0;
        }

        // the object prefix table's place
        float* po;
        if constexpr (MODE == kArena) {
            const unsigned int need4 = (unsigned int)((fmax - fmin + 1) * (po_row_floats(H) / 4));
            if (own4 < need4) {
                if (tid == 0) {
                    const Const<ChainArgs> A = again(a);
                    place = arena_take(A->room4, need4, full, [&](unsigned int n) {
                        return atomicAdd(&A->head->used4, n);
                    });
                    if (place == kNoPlace) A->rest[atomicAdd(&A->head->nrest, 1u)] = col;
                }
                __syncthreads();
                const unsigned int at = (unsigned int)__builtin_amdgcn_readfirstlane((int)place);
                full = at == kNoPlace;
                if (!full) {
                    own = at;
                    own4 = need4;
                }
                __syncthreads();                 // before the next column writes place
                if (full) continue;
            }
            po = again(a)->po + (size_t)own * 4;
        } else {
            const Const<ChainArgs> A = again(a);
            po = A->po + (size_t)(MODE == kFrame ? col : (int)blockIdx.x) * (size_t)A->stride;
        }

        // Sec. 4.2: the small tables by the first five waves, the thresholds by
        // all, the object rows by whoever is free
        for (int t = wave; t < 5; t += nw) {
            float* const dst = reinterpret_cast<float*>(t == 0 || t == 1 || t == 4 ? L.pre : L.base) +
                               (t == 0 || t == 2 ? 0 : (t == 4 ? 2 : 1));
            float* out = nullptr;
            if constexpr (MODE == kFrame) {
                if (a->ex.prefix && t < 4)
                    out = a->ex.prefix + ((size_t)t * a->job.ncols + col) * stride;
            }
            small_table(again(job_at), qs, t, dst, out);
        }
        const int32_t *const fg_hi = again(job_at)->fg_hi, *const fg_lo = again(job_at)->fg_lo;
        for (int b = tid; b <= H; b += nt) {
            const int r = max(H - 1 - b, 0);
            L.base[b].z = __builtin_bit_cast(float, fg_hi[r]);
            L.base[b].w = __builtin_bit_cast(float, fg_lo[r]);
        }
        if constexpr (MODE == kFrame) {
            if (a->ex.range && tid == 0) {
                a->ex.range[2 * col] = fmin;
                a->ex.range[2 * col + 1] = fmax;
            }
        }
#ifdef STX_PHASE_TIMING
        t2 = __builtin_amdgcn_s_memtime();
#endif
        float* const stg = stage + wave * (kMaxDisparity + 4);
        if (H <= 256) object_rows<1>(again(job_at), qs, stg, edges, &red[3], po, fmin, fmax);
        else if (H <= 512) object_rows<2>(again(job_at), qs, stg, edges, &red[3], po, fmin, fmax);
        else object_rows<4>(again(job_at), qs, stg, edges, &red[3], po, fmin, fmax);
        __syncthreads();

        // Sec. 4.3-4.4
        const Const<JobDesc> Jc = again(job_at);
        const Prior prior = load_const(&Jc->prior);
        const ChainCol c = chain_column(H, Jc->vtop, prior, po + 3, fmin, fmax,
                                        (uint32_t)po_row_floats(H) * 4u);
        if (H > 64) {
            chain_bounds(c, L, wave, nw);
            __syncthreads();
        }
#ifdef STX_PHASE_TIMING
        t3 = __builtin_amdgcn_s_memtime();
#endif
        chain_solve(c, L, prior, [&]() {
#ifdef STX_PHASE_TIMING
            t4 = __builtin_amdgcn_s_memtime();
#endif
            const Const<JobDesc> J = again(job_at);
            ColumnOut out;
            out.count = J->counts + col;
            out.rec = J->records + (size_t)col * J->cap * 3;
            out.total = J->total + col;
            out.overflow = J->overflow + col;
            out.cap = J->cap;
            return out;
        });
#ifdef STX_PHASE_TIMING
        if (tid == 0) {
            __builtin_amdgcn_s_waitcnt(0);
            phase_add(kPhaseReduce, t1 - t0);
            phase_add(kPhaseScans, t2 - t1);
            phase_add(kPhaseObjectTable, t3 - t2);
            phase_add(kPhaseRecurrence, t4 - t3);
            phase_add(kPhaseBacktrack, __builtin_amdgcn_s_memtime() - t4);
            phase_add(kPhaseTasks, 1ull);
        }
#endif
        if constexpr (MODE != kFrame) __syncthreads();   // the next column reuses it all
    }
#ifdef STX_PHASE_TIMING
    phase_add(kPhaseLifetime, __builtin_amdgcn_s_memtime() - t_entry);
#endif
}

namespace {

__global__ void arena_reset_kernel(ArenaHead* h) { *h = ArenaHead{0u, 0u, 0u, 0u}; }

template <int MODE>
hipError_t start(const ChainArgs& a, int grid, int waves, int lds, hipStream_t st) {
    hipLaunchKernelGGL(chain_frame_kernel<MODE>, dim3((unsigned)grid), dim3(64u * (unsigned)waves),
                       (size_t)lds, st, a);
    return hipGetLastError();
}

// A workgroup has 16 waves where there is a compute unit for each, else 8, two
// to a compute unit (2048x880, 409 columns: 242 us with 16 waves, 201 with 8, at
// the same stage of the kernel), as long as their LDS lets two in: a frame's
// columns up to 889 rows, others up to 888.  Above, one is there whatever its
// waves, and has 16: 8 / 16 waves on frames of 2048 columns' width and 256
// disparities took, with 3-pixel columns, 388 / 346 us at 896 rows and 468 / 413
// at 1024 (889 rows: two of 8 waves 314, one of 16 340), 16 frames at once 5,466 /
// 4,817 at 889 and 6,546 / 5,523 at 1024.  Four halves of a group's gathers in
// flight instead of two groups' would let three workgroups of 8 in (80 registers
// a lane): 16 frames 1024x440 took 508 us instead of 476, one frame 96 instead of
// 78.
int frame_waves_of(int ncols, int H, int D, int num_cu, bool frame) {
    const int few = chain_waves(H, 8);
    const bool alone = ncols <= num_cu ||
                       chain_resident(few, lds_bytes(H, D, few) + static_lds(frame)) < 2;
    return alone ? chain_waves(H, 16) : few;
}

constexpr size_t kHeadBytes = 256;
size_t round256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

hipError_t launch_chain_frame(const JobDesc& job, float* po, const ChainExports& ex, int num_cu,
                              hipStream_t st) {
    ChainArgs a{};
    a.job = job;
    a.ex = ex;
    a.po = po;
    a.stride = (long long)chain_table_floats(job.H, job.D);
    const int nw = frame_waves_of(job.ncols, job.H, job.D, num_cu, true);
    return start<kFrame>(a, job.ncols, nw, lds_bytes(job.H, job.D, nw), st);
}

size_t chain_arena_bytes(int ncols, int H, int D, int tables) {
    return kHeadBytes + round256(sizeof(int) * (size_t)ncols) +
           chain_table_floats(H, D) * sizeof(float) * (size_t)tables + kTableGuardBytes;
}

// A frame whose tables all fit is launched like any other, 1.1 to 9 times as
// fast as a wave per column.  In a shared workspace the resident workgroups take
// columns in turn, with a task and a place handed out and barriers around each
// (64 rows and bins: 41 us a column, 21 in a launch with a workgroup each), and of
// few rows and disparities a wave takes less.  Spread / a wave per column, us, rows
// x bins, columns: 32x256 4,096 150 / 98; 64x128 4,096 166 / 119; 96x128
// 2,048 128 / 126, 8,192 407 / 349; 128x64 8,192 424 / 271; 64x256 2,048 92 / 103,
// 4,096 168 / 165, 8,192 368 / 290; 128x128 2,048 147 / 156, 4,096 257 / 249, 8,192
// 532 / 440; 192x128 8,192 768 / 941; 96x256 8,192 459 / 670; 440x128 4,096 921 /
// 3,267.
bool chain_arena_pays(int ncols, int H, int D, size_t ws_bytes, int num_cu) {
    const int cells = H * D;
    return chain_arena_bytes(ncols, H, D, ncols) <= ws_bytes ||
           cells > (ncols > 16 * num_cu ? 16384 : 12288);
}

hipError_t launch_chain_arena(const JobDesc& job, void* ws, size_t ws_bytes, int num_cu,
                              hipStream_t st) {
    const size_t base = chain_arena_bytes(job.ncols, job.H, job.D, 0);
    const size_t table = chain_table_floats(job.H, job.D) * sizeof(float);
    if (job.ncols < 1 || ws_bytes < base + table) return hipErrorInvalidValue;
    char* const p = static_cast<char*>(ws);
    float* const po = reinterpret_cast<float*>(p + base - kTableGuardBytes);
    const size_t tables = (ws_bytes - base) / table;
    // room for every column's largest table: a frame like any other
    if (tables >= (size_t)job.ncols) return launch_chain_frame(job, po, ChainExports{}, num_cu, st);
    // otherwise columns take what their own disparity range needs; those for
    // which nothing is left run afterwards, with a whole table each
    ChainArgs a{};
    a.job = job;
    a.head = reinterpret_cast<ArenaHead*>(p);
    a.rest = reinterpret_cast<int*>(p + kHeadBytes);
    a.po = po;
    a.stride = (long long)chain_table_floats(job.H, job.D);
    a.room4 = (unsigned int)((ws_bytes - base) / 16);
    hipLaunchKernelGGL(arena_reset_kernel, dim3(1), dim3(1), 0, st, a.head);
    hipError_t e = hipGetLastError();
    const int nw = frame_waves_of(job.ncols, job.H, job.D, num_cu, false);
    const int lds = lds_bytes(job.H, job.D, nw);
    const int per_cu = chain_resident(nw, lds + static_lds(false));
    if (e == hipSuccess) e = start<kArena>(a, std::min(job.ncols, per_cu * num_cu), nw, lds, st);
    if (e == hipSuccess)
        e = start<kArenaRest>(a, (int)std::min<size_t>(tables, (size_t)std::min(job.ncols, num_cu)),
                              nw, lds, st);
    return e;
}

int chain_batch_waves(int hmax, int ntasks, int num_cu) {
    return frame_waves_of(ntasks, hmax, kMaxDisparity, num_cu, false);
}
int chain_batch_per_cu(int hmax, int waves) {
    return chain_resident(waves, lds_bytes(hmax, kMaxDisparity, waves) + static_lds(false));
}

hipError_t launch_chain_batch(const JobDesc* jobs, const int2* tasks, int ntasks,
                              unsigned int* counter, float* scratch, long long stride, int hmax,
                              int grid, int waves, hipStream_t st) {
    ChainArgs a{};
    a.jobs = jobs;
    a.tasks = tasks;
    a.ntasks = ntasks;
    a.counter = counter;
    a.po = scratch;
    a.stride = stride;
    return start<kBatch>(a, grid, waves, lds_bytes(hmax, kMaxDisparity, waves), st);
}

hipError_t chain_frame_setup(int lds_per_block) {
    hipError_t e = hipSuccess;
    // the static LDS of the kernels comes out of the same budget
    const int dyn = lds_per_block - 256;
    for (const void* f : {reinterpret_cast<const void*>(&chain_frame_kernel<kFrame>),
                          reinterpret_cast<const void*>(&chain_frame_kernel<kBatch>),
                          reinterpret_cast<const void*>(&chain_frame_kernel<kArena>),
                          reinterpret_cast<const void*>(&chain_frame_kernel<kArenaRest>)})
        if (e == hipSuccess)
            e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, dyn);
    return e;
}

}  // namespace stx::persist
