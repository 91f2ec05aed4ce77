// resident.hip -- Algorithm 1 (Section 2) with the messages held on the chip.
//
// Up to kResMaxN points, S, R and A of a solve (12 bytes per element) fit in
// the vector registers of the compute units (128 MB), so one launch of
// workgroups that all run at once runs the whole solve: the matrices are read once and written once,
// and an iteration moves only column vectors between workgroups.  The
// streaming passes (ap_iter.hip) take two launches and 20 bytes per element
// and iteration: 13.8 us at n = 500, 29 at 2000, 49 at 3001; here an
// iteration takes 4.9, 8.7 and 13.5 us.  About 4 us of that are the two
// exchanges between the workgroups (two round trips to device-coherent
// memory each), the rest is vector arithmetic (20 instructions per element).
//
// A member (workgroup) owns a block of rows.  A wavefront holds whole rows:
// lane l has the columns 4 (64 j + l) .. + 3 of chunk j, so the top-2 of a
// row is a wavefront reduction and no barrier is needed per row.  Between
// iterations
//   1. max(0, r) of the block goes to LDS, every thread adds up columns in
//      row order and publishes the member's column sums to the member that
//      owns the column's row (exchange 1),
//   2. the owners add the members' sums (FP64, member order), form t_k and
//      c_k and publish t_k with the row's exemplar flag to everyone
//      (exchange 2), which also gives every member the stop rule's counts.
// The published words carry their own iteration: a column sum is
// non-negative, so its sign bit alternates each time its slot is reused;
// t_k travels with a 32-bit stamp in one 8-byte word.  A reader polls the
// data itself: no flag, no fence and no cache write-back is needed, only
// device-scope accesses to the exchanged words.  Two slots per word (by
// iteration parity) are enough, since a member can publish iteration t + 2
// only after every owner has read iteration t.
//
// The sums are those of the streaming passes: rows are grouped as there (at
// most 512 groups of consecutive rows, each summed in FP32 in row order) and
// the groups are added in FP64, so results agree with the launched passes.
#include <atomic>
#include <cmath>
#include <condition_variable>
#include <cstring>
#include <mutex>

#include "apx_internal.h"

namespace apx {
namespace {

constexpr float kNegInf = -INFINITY;
// (chunks, rows per wavefront) instantiated.  The 168 registers of a lane hold
// eight chunks of three matrices without a spill; above, chunks of S lie in LDS
// (below) and 12, 36, 48 and 100 bytes per lane (9 to 12 chunks) still go
// through scratch.  The variants of a batch's kernel share one allocation, so a
// batch launches three classes of sizes apart: 1 to 4, 5 to 8 and 9 to 12
// chunks (20, 0 and 168 bytes; with the two upper ones in one kernel, its
// tables in vector registers, 444: 16 instances of 1500 points 7.6 ms, 7.1
// now, 4 of 2800 5.76 and 5.46).
#define APX_RES_CLASS0(X) \
    X(1, 1) X(1, 2) X(1, 3) X(1, 5) X(2, 1) X(2, 2) X(2, 3) X(3, 1) X(3, 2) X(4, 1) X(4, 2)
#define APX_RES_CLASS1(X) X(5, 1) X(6, 1) X(7, 1) X(8, 1)
#define APX_RES_CLASS2(X) X(9, 1) X(10, 1) X(11, 1) X(12, 1)
#define APX_RES_VARIANTS(X) APX_RES_CLASS0(X) APX_RES_CLASS1(X) APX_RES_CLASS2(X)
constexpr int kClassChunks = 4;

constexpr int RW = kResWaves;     // wavefronts per workgroup (3 per SIMD: 168 registers)
constexpr int RT = 64 * RW;
// Up to 1536 points (groups of at most three rows) a column sum reads four
// rows at once and looks up the ends of groups in a mask (the sum of 24 rows
// at n = 750 3780 -> 2500 cycles); longer groups are summed one by one (n =
// 3001: 13.5 us per iteration, 14.8 with the mask).
constexpr int kSmallGroups = 6;
constexpr int kRedLanes = 8;      // lanes that finish one column's sum
constexpr int kMaxRows = 64;      // rows a member can own (one bit each, kRedLanes threads each)
static_assert(kMaxRows * kRedLanes <= RT, "threads of the reduction");
// Polls of one word before a wait is given up (each takes about a
// microsecond; a legitimate wait is one iteration of another member).
constexpr uint32_t kPollLimit = 1u << 21;
// Until the members have met once, one of them may not run at all: other work
// holds its compute unit, which may itself be waiting for this one to end (a
// solve of another process).  That wait is short, since giving up is cheap
// there: nothing has been written and the launched passes need no company.
constexpr uint32_t kMeetLimit = 1u << 12;
// A batch's workgroups have all met when they wait for earlier instances.
constexpr uint32_t kArriveLimit = 1u << 28;

typedef unsigned long long u64;
typedef float v4f __attribute__((ext_vector_type(4)));

// Global-memory views of the pointers of an instance (read from memory, so
// the compiler would take them as generic).
#define APX_GLOBAL __attribute__((address_space(1)))
__device__ __forceinline__ u64 ld_dev(const u64 *p) {
    return __hip_atomic_load((const APX_GLOBAL u64 *)p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void st_dev(u64 *p, u64 v) {
    __hip_atomic_store((APX_GLOBAL u64 *)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// ... at a 32-bit word offset from a uniform base (one address register)
__device__ __forceinline__ u64 ld_dev(const u64 *p, uint32_t w) {
    return ld_dev(reinterpret_cast<const u64 *>(reinterpret_cast<const char *>(p) + (u64)(w * 8u)));
}
__device__ __forceinline__ void st_dev(u64 *p, uint32_t w, u64 v) {
    st_dev(reinterpret_cast<u64 *>(reinterpret_cast<char *>(p) + (u64)(w * 8u)), v);
}
__device__ __forceinline__ v4f ld_row(const float *p) { return *(const APX_GLOBAL v4f *)p; }
__device__ __forceinline__ void st_row(float *p, v4f v) { *(APX_GLOBAL v4f *)p = v; }
__device__ __forceinline__ float ld_one(const float *p) { return *(const APX_GLOBAL float *)p; }
__device__ __forceinline__ void st_one(float *p, float v) { *(APX_GLOBAL float *)p = v; }

// max(0, x), min(0, x) and max(a, b) as single instructions (the library
// functions quiet a signalling NaN first, one more instruction per element).
// Of a number and a NaN all three give the number, like fmaxf and fminf: with
// similarities of -inf a column sum can be +inf and t_k - max(0, r) then NaN.
// minf is only for values that are no NaN.
__device__ __forceinline__ float max0(float x) {
    float y;
    asm("v_max_f32 %0, 0, %1" : "=v"(y) : "v"(x));
    return y;
}
__device__ __forceinline__ float min0(float x) {
    float y;
    asm("v_min_f32 %0, 0, %1" : "=v"(y) : "v"(x));
    return y;
}
__device__ __forceinline__ float maxf(float a, float b) { return __builtin_amdgcn_fmed3f(a, b, INFINITY); }
__device__ __forceinline__ float minf(float a, float b) { return __builtin_amdgcn_fmed3f(a, b, -INFINITY); }

template <int CTRL, int RM = 0xF>
__device__ __forceinline__ float dpp(float x) {
    return __int_as_float(
        __builtin_amdgcn_update_dpp(__float_as_int(kNegInf), __float_as_int(x), CTRL, RM, 0xF, false));
}
template <int CTRL, int RM = 0xF>
__device__ __forceinline__ void top2_step(float &v1, float &v2) {
    const float o1 = dpp<CTRL, RM>(v1), o2 = dpp<CTRL, RM>(v2);
    v2 = maxf(maxf(v2, o2), minf(v1, o1));
    v1 = maxf(v1, o1);
}
__device__ __forceinline__ float lane63(float x) {
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 63));
}
__device__ __forceinline__ float lane0(float x) {
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x)));
}
// The two largest of all lanes' (v1, v2); quad swaps, half-row and row
// mirrors, then the row broadcasts of lanes 15 and 31.
__device__ __forceinline__ void wave_top2(float &v1, float &v2) {
    top2_step<0xB1>(v1, v2);
    top2_step<0x4E>(v1, v2);
    top2_step<0x141>(v1, v2);
    top2_step<0x140>(v1, v2);
    top2_step<0x142, 0xA>(v1, v2);
    top2_step<0x143, 0xC>(v1, v2);
    v1 = lane63(v1);
    v2 = lane63(v2);
}
__device__ __forceinline__ float wave_max(float x) {
    x = maxf(x, dpp<0xB1>(x));
    x = maxf(x, dpp<0x4E>(x));
    x = maxf(x, dpp<0x141>(x));
    x = maxf(x, dpp<0x140>(x));
    x = maxf(x, dpp<0x142, 0xA>(x));
    x = maxf(x, dpp<0x143, 0xC>(x));
    return lane63(x);
}

// Keeps the compiler from holding a value derived from x across this point
// (a + s of a whole row would take as many registers as a matrix).
__device__ __forceinline__ void opaque(float &x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void opaque(int &x) { asm volatile("" : "+v"(x)); }

// First row of group g of G: G = n (a group is a row) or G = 512.
__device__ __forceinline__ int group_row(int g, int n, int G) { return G == n ? g : (int)(((uint32_t)g * n) >> 9); }
__device__ __forceinline__ int group_of(int k, int n, int G) {
    return G == n ? k : (int)((((uint32_t)k + 1u) * 512u - 1u) / (uint32_t)n);
}

// Above 9 chunks the registers do not hold all three matrices: max(0, r) is
// then summed in two parts of the columns, and the LDS freed holds chunks of
// S (at 12 chunks six: 44 registers spill; without it 72, and an iteration at
// n = 3001 took 21 us instead of 13.5).
constexpr int res_s_chunks(int ej) { return ej <= 9 ? 0 : ej == 10 ? 3 : 6; }
constexpr int res_parts(int ej) { return ej <= 9 ? 1 : 2; }

// LDS of a workgroup: max(0, r) of its rows, the column vector t (which the
// reduction of exchange 1 uses while t is dead), small per-row values.
struct ResLds {
    float *pos;       // [rows][columns of a part]
    float *s;         // [rows][columns of S held here]
    float *t;         // [256 EJ]
    double *red;      // aliases t: [slices][rows]
    float *c;         // c_k of the member's rows
    float *rdiag;     // r(k,k) of the member's rows
    int *e;           // exemplar flags of the member's rows
    int *cnt;         // [2][2]: exemplars, changed flags
    int *fail;
    uint32_t *limit;  // polls of the exchanges' waits, and the iteration that gives them
    int *give_up;     // up (not in registers: the rows need them)
};

struct ResArgs {
    ResInst one;              // the instance of a single solve (workgroup = member)
    const ResInst *insts;     // a batch's instances
    const ResTask *tasks;     // workgroup b runs tasks [lane[b], lane[b+1]) in order
    const int32_t *lane;
    u64 *abort;               // a batch's words: [0] set when a wait was given up, [1] workgroups that run
    int32_t give_up;          // iteration whose waits are given up at once (none: -1; kGiveUpAtEnd: the labels')
    float lam, lam0;          // damping; damping of the first responsibility step
    int32_t max_iter, conv_iter;
};

// One member's part of a solve: EJ float4 chunks per lane and row, up to RPW
// rows per wavefront.  False (in every thread) when a wait was given up.
template <int EJ, int RPW>
__device__ __forceinline__ bool res_run(const ResInst &d, int rank, const ResArgs &p, char *lds) {
#pragma clang fp contract(off)
    constexpr int NC = 256 * EJ;              // columns held, padding included
    constexpr int SL = res_s_chunks(EJ);      // chunks of S held in LDS
    constexpr int SR = EJ - SL;               // ... in registers
    constexpr int NH = res_parts(EJ);         // parts of max(0, r)
    constexpr int HC = (EJ + NH - 1) / NH;    // chunks of a part
    constexpr int PC = 256 * HC;              // columns of a part
    // (opaque: what follows from the thread's index would be held across a
    // batch's instances, beside the rows)
    int tid0 = (int)threadIdx.x;
    opaque(tid0);
    const int tid = tid0, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = d.n, G = d.groups, M = d.members;
    const int g0 = rank * d.gpm;
    const int g1 = g0 + d.gpm < G ? g0 + d.gpm : G;
    const int row0 = group_row(g0, n, G), rows = group_row(g1, n, G) - row0;

    ResLds L;
    L.t = reinterpret_cast<float *>(lds);
    L.red = reinterpret_cast<double *>(lds);
    constexpr int tw = NC * 4 > RT * 8 ? NC * 4 : RT * 8;
    L.c = reinterpret_cast<float *>(lds + tw);
    L.rdiag = L.c + kMaxRows;
    L.e = reinterpret_cast<int *>(L.rdiag + kMaxRows);
    L.cnt = L.e + kMaxRows;
    L.fail = L.cnt + 4;
    L.limit = reinterpret_cast<uint32_t *>(L.fail + 1);
    L.give_up = L.fail + 2;
    L.pos = reinterpret_cast<float *>(lds + tw + 3 * 4 * kMaxRows + 32);
    L.s = L.pos + rows * PC;

    // ---- the member's rows into registers.  The diagonal is kept apart; its
    // place and the padding columns hold s = r = -inf, which never wins a
    // maximum and adds nothing to a column.  A step of damping 0 makes their r
    // 0 * -inf = NaN (with damping 0, or the first step from column-structured
    // availabilities): max0 and maxf then give the other operand, as for a
    // message that is NaN itself, no comparison with it holds, and it is never
    // stored.
    float s[RPW][SR][4], r[RPW][EJ][4], a[RPW][EJ][4];
    float sd[RPW], rd[RPW], ad[RPW];
#pragma unroll
    for (int q = 0; q < RPW; ++q) {
        const int lr = wave + q * RW, i = row0 + lr;
        sd[q] = rd[q] = ad[q] = 0.0f;
#pragma unroll
        for (int j = 0; j < EJ; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (j < SR) s[q][j < SR ? j : 0][e] = kNegInf;
                r[q][j][e] = kNegInf;
                a[q][j][e] = 0.0f;
            }
        if (lr >= rows) continue;
        const int64_t at = (int64_t)i * d.ld;
#pragma unroll
        for (int j = 0; j < EJ; ++j) {
            const int c = 4 * (64 * j + lane);
            if (j >= SR) {
                v4f sv = {kNegInf, kNegInf, kNegInf, kNegInf};
                if (c < n) {
                    const v4f g = ld_row(d.S + at + c);
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (c + e < n && c + e != i) sv[e] = g[e];
                }
                *reinterpret_cast<v4f *>(L.s + lr * (256 * SL) + 4 * (64 * (j - SR) + lane)) = sv;
            }
            if (c >= n) continue;
            v4f sv = {kNegInf, kNegInf, kNegInf, kNegInf};
            if (j < SR) sv = ld_row(d.S + at + c);
            v4f rv = {0.f, 0.f, 0.f, 0.f}, av = rv;
            if (d.load_a) av = ld_row(d.A + at + c);
            if (d.load_r) rv = ld_row(d.R + at + c);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (c + e < n && c + e != i) {
                    if (j < SR) s[q][j < SR ? j : 0][e] = sv[e];
                    r[q][j][e] = rv[e];
                    a[q][j][e] = av[e];
                }
            __builtin_amdgcn_sched_barrier(0);
        }
        sd[q] = ld_one(d.S + at + i);
        if (d.load_a) ad[q] = ld_one(d.A + at + i);
        if (d.load_r) rd[q] = ld_one(d.R + at + i);
    }

    // chunk j of a row of S
    auto get_s = [&](int q, int lr, int j) -> v4f {
        if (j < SR) return v4f{s[q][j][0], s[q][j][1], s[q][j][2], s[q][j][3]};
        return *reinterpret_cast<const v4f *>(L.s + lr * (256 * SL) + 4 * (64 * (j - SR) + lane));
    };

    // ---- this thread's columns in exchange 1: columns tid + u RT of each part
    constexpr int NU = (NC + RT - 1) / RT, NP = (PC + RT - 1) / RT;
    uint32_t poff[NH][NP];
#pragma unroll
    for (int h = 0; h < NH; ++h)
#pragma unroll
    for (int u = 0; u < NP; ++u) {
        const int k = h * PC + tid + u * RT;
        poff[h][u] = 0;
        if (tid + u * RT < PC && k < n) {
            const int b = group_of(k, n, G) / d.gpm;
            const int bg = (b + 1) * d.gpm;
            const int b0 = group_row(b * d.gpm, n, G), b1 = group_row(bg < G ? bg : G, n, G);
            poff[h][u] = (uint32_t)(b0 * M + rank * (b1 - b0) + (k - b0));
        }
    }
    const int64_t pstride = (int64_t)n * M;
    u64 ends = 0ull;       // bit r: row r of the block is the last of its group
    for (int g = g0; g < g1; ++g) ends |= 1ull << (group_row(g + 1, n, G) - row0 - 1);
    const int slices = RT / rows;
    int rsc = (tid / rows) << 16 | (tid % rows);   // slice and column of this thread in exchange 1

    // At t = 0 the availability step leaves A_0 as it is: t = +inf makes its
    // update min(0, t - max(0, r)) zero whatever R_0 holds.
    for (int k = tid; k < NC; k += RT) L.t[k] = INFINITY;
    for (int k = tid; k < kMaxRows; k += RT) {
        L.e[k] = 0;
        L.c[k] = 0.0f;
    }
    if (tid < 4) L.cnt[tid] = 0;
    if (tid == 0) {
        *L.fail = 0;
        *L.limit = kMeetLimit;
        *L.give_up = p.give_up;
    }
    uint32_t eprev = 0u;   // flags of this thread's columns in the last iteration
    int run = 0;
    const float lam = p.lam, oml = 1.0f - lam;
    float lu = p.lam0, lo = 1.0f - p.lam0;    // damping of the next responsibility step
    float la = 1.0f, oa = 0.0f;               // ... availability step: A_0 stays as it is at t = 0
    bool converged = false;
    int t = 0;
    __syncthreads();

    for (;; ++t) {
        // ---- A_t (t >= 1), the exemplar decision, the top-2 of a + s
        float v1[RPW], v2[RPW], vd[RPW];
        int ex[RPW];
#pragma unroll
        for (int q = 0; q < RPW; ++q) {
            // Opaque: v_med3 of (v1, v2, NaN) is v2, but with a v2 known to be
            // -inf the compiler makes it a minimum of v1 and NaN, which is v1.
            v1[q] = v2[q] = kNegInf;
            opaque(v2[q]);
        }
        {
            float dv[RPW], D[RPW];
#pragma unroll
            for (int q = 0; q < RPW; ++q) {
                const int lr = wave + q * RW;
                ad[q] = la * ad[q] + oa * L.c[lr < rows ? lr : 0];
                D[q] = ad[q] + rd[q];
                dv[q] = kNegInf;
            }
#pragma unroll
            for (int j = 0; j < EJ; ++j) {
                const v4f t4 = *reinterpret_cast<const v4f *>(L.t + 4 * (64 * j + lane));
#pragma unroll
                for (int q = 0; q < RPW; ++q) {
                    const int lr = wave + q * RW;
                    const v4f s4 = get_s(q, lr < rows ? lr : 0, j);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float x = r[q][j][e];
                        const float upd = min0(t4[e] - max0(x));
                        const float an = la * a[q][j][e] + oa * upd;
                        a[q][j][e] = an;
                        dv[q] = maxf(dv[q], an + x);
                        const float v = an + s4[e];
                        v2[q] = __builtin_amdgcn_fmed3f(v1[q], v2[q], v);
                        v1[q] = maxf(v1[q], v);
                    }
                }
                // one chunk at a time: the next chunks' t would take the registers
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int q = 0; q < RPW; ++q) {
                const float w = wave_max(dv[q]);
                const float dq = lane0(D[q]);
                bool is = w < dq;
                if (w == dq && dq > kNegInf) {
                    // a tie goes to the lowest column: an exemplar unless a lower one reaches D
                    const int i = row0 + wave + q * RW;
                    bool lower = false;
                    int ln = lane;
                    opaque(ln);
#pragma unroll
                    for (int j = 0; j < EJ; ++j)
#pragma unroll
                        for (int e = 0; e < 4; ++e) {
                            opaque(r[q][j][e]);
                            lower |= 4 * (64 * j + ln) + e < i && a[q][j][e] + r[q][j][e] == dq;
                        }
                    is = !__any(lower);
                }
                ex[q] = is && t > 0;
            }
        }
#pragma unroll
        for (int q = 0; q < RPW; ++q) {
            wave_top2(v1[q], v2[q]);
            vd[q] = ad[q] + sd[q];
            v2[q] = __builtin_amdgcn_fmed3f(v1[q], v2[q], vd[q]);
            v1[q] = maxf(v1[q], vd[q]);
        }

        // ---- where the stop rule can fire, its counts are needed before R_t
        // is overwritten: each member publishes its own, everyone adds them
        if (t > 0 && (t >= p.max_iter || (p.conv_iter > 0 && run + 1 >= p.conv_iter))) {
#pragma unroll
            for (int q = 0; q < RPW; ++q) {
                const int lr = wave + q * RW;
                if (lane == 0 && lr < rows) {
                    if (ex[q]) atomicAdd(&L.cnt[2], 1);
                    if (ex[q] != L.e[lr]) atomicOr(&L.cnt[3], 1);
                }
            }
            __syncthreads();
            if (tid == 0)
                st_dev(d.stat + rank, ((u64)(uint32_t)t << 32) | ((u64)L.cnt[3] << 16) | (u64)L.cnt[2]);
            u64 w = 0ull;
            for (int m = tid; m < M; m += RT) {
                uint32_t polls = 0u;
                while ((uint32_t)((w = ld_dev(d.stat + m)) >> 32) != (uint32_t)t)
                    if (++polls > kPollLimit) {
                        *L.fail = 1;
                        break;
                    }
            }
            // (M <= RT: at most one word per thread)
            __syncthreads();
            if (tid == 0) L.cnt[2] = L.cnt[3] = 0;
            __syncthreads();
            if (tid < M) {
                atomicAdd(&L.cnt[2], (int)(w & 0xFFFFu));
                if (w & 0x10000u) atomicOr(&L.cnt[3], 1);
            }
            __syncthreads();
            const int nex = L.cnt[2], changed = L.cnt[3];
            if (*L.fail) return false;
            __syncthreads();
            if (tid == 0) L.cnt[2] = L.cnt[3] = 0;
            const int now = (t > 1 && !changed) ? run + 1 : 1;
            converged = p.conv_iter > 0 && now >= p.conv_iter && nex > 0;
            if (converged || t >= p.max_iter) {
#pragma unroll
                for (int q = 0; q < RPW; ++q) {
                    const int lr = wave + q * RW;
                    if (lane == 0 && lr < rows) L.e[lr] = ex[q];
                }
                break;
            }
            __syncthreads();
        }

        // ---- R_{t+1} (Eq. (2), damped).  The largest column takes the second
        // value; under a tie the two are equal, so "a + s is the largest" names it.
        // max(0, r) goes to LDS one part of the columns at a time; its column
        // sums follow, group by group (with one member they are the totals).
        // What these phases derive from the thread's index is formed anew in
        // each iteration: the rows need the registers.
        const bool first = t == 0;
        const int par = t & 1;
        const u64 sign = (u64)(((t >> 1) & 1) ^ 1) << 63;
        u64 *part = d.part + par * pstride;
        int tid = (int)threadIdx.x;
        opaque(tid);
        opaque(rsc);
#pragma unroll
        for (int h = 0; h < NH; ++h) {
            if (h > 0) __syncthreads();       // the sums of the part before have read it
#pragma unroll
            for (int q = 0; q < RPW; ++q) {
                const int lr = wave + q * RW;
                if (lr >= rows) continue;
                const float m_other = lo * v1[q], m_self = lo * v2[q];
#pragma unroll
                for (int j = h * HC; j < (h + 1) * HC && j < EJ; ++j) {
                    const v4f s4 = get_s(q, lr, j);
                    v4f x;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        opaque(a[q][j][e]);
                        const float m = a[q][j][e] + s4[e] == v1[q] ? m_self : m_other;
                        const float rn = (lu * r[q][j][e] + lo * s4[e]) - m;
                        r[q][j][e] = rn;
                        x[e] = max0(rn);
                    }
                    *reinterpret_cast<v4f *>(L.pos + lr * PC + 4 * (64 * (j - h * HC) + lane)) = x;
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (h == NH - 1) {
                    rd[q] = (lu * rd[q] + lo * sd[q]) - (vd[q] == v1[q] ? m_self : m_other);
                    if (lane == 0) {
                        L.rdiag[lr] = rd[q];
                        L.e[lr] = ex[q];
                    }
                }
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < NP; ++u) {
                const int kp = tid + u * RT, k = h * PC + kp;
                if (kp < PC && k < n) {
                    double tot = 0.0;
                    if constexpr (EJ <= kSmallGroups) {
                        // groups of one to three rows: four rows in flight
                        float acc = 0.0f;
                        for (int lr = 0; lr < rows; lr += 4) {
                            float v[4];
#pragma unroll
                            for (int x = 0; x < 4; ++x) v[x] = L.pos[(lr + x < rows ? lr + x : lr) * PC + kp];
#pragma unroll
                            for (int x = 0; x < 4; ++x) {
                                if (lr + x < rows) acc += v[x];
                                if ((ends >> (lr + x)) & 1ull) {
                                    tot += (double)acc;
                                    acc = 0.0f;
                                }
                            }
                        }
                    } else {
                        int lr = 0;
                        for (int g = g0; g < g1; ++g) {
                            const int end = group_row(g + 1, n, G) - row0;
                            float acc = 0.0f;
                            for (; lr < end; ++lr) acc += L.pos[lr * PC + kp];
                            tot += (double)acc;
                        }
                    }
                    if (M > 1) {
                        st_dev(part, poff[h][u], ((u64)__double_as_longlong(tot) & 0x7FFFFFFFFFFFFFFFull) | sign);
                    } else {
                        L.t[k] = (float)((double)L.rdiag[k] + tot);
                        L.c[k] = (float)tot;
                    }
                }
            }
        }
        lu = la = lam;
        lo = oa = oml;
        const int nu = t & 1;             // counters of this iteration
        if (M > 1) {
            // exchange 1: the members' sums of this member's columns
            double sum = 0.0;
            bool bad = false;
            const int rsl = rsc >> 16, rcol = rsc & 0xFFFF;
            if (rsl < slices) {
                const u64 *src = part + (int64_t)row0 * M;
                for (int m = rsl; m < M; m += 4 * slices) {
                    u64 w[4];
                    uint32_t polls = 0u;
                    for (;;) {
                        u64 off = 0ull;    // sign bit set: a word is not this iteration's
#pragma unroll
                        for (int x = 0; x < 4; ++x) {
                            const int mm = m + x * slices;
                            w[x] = sign;
                            if (mm < M) w[x] = ld_dev(src, (uint32_t)(mm * rows + rcol));
                        }
#pragma unroll
                        for (int x = 0; x < 4; ++x) off |= w[x] ^ sign;
                        if ((long long)off >= 0) break;
                        if (++polls > *L.limit) {
                            bad = true;
                            break;
                        }
                    }
#pragma unroll
                    for (int x = 0; x < 4; ++x)
                        if (m + x * slices < M) sum += __longlong_as_double((long long)(w[x] & 0x7FFFFFFFFFFFFFFFull));
                }
                L.red[rsl * rows + rcol] = sum;
            }
            if (bad) *L.fail = 1;
            __syncthreads();
            const int lr = tid / kRedLanes, l = tid & (kRedLanes - 1);
            if (lr < rows) {
                double tot = 0.0;
                for (int x = l; x < slices; x += kRedLanes) tot += L.red[x * rows + lr];
#pragma unroll
                for (int o = 1; o < kRedLanes; o <<= 1) tot += __shfl_xor(tot, o, 64);
                if (l == 0) {
                    const float tf = (float)((double)L.rdiag[lr] + tot);
                    L.c[lr] = (float)tot;
                    st_dev(d.pair + (int64_t)par * n + row0, (uint32_t)lr,
                           ((u64)(((uint32_t)(t + 1) << 1) | (uint32_t)L.e[lr]) << 32) | __float_as_uint(tf));
                }
            }
            __syncthreads();              // the sums have been read: t may be written over them
            // exchange 2: t_k and the exemplar flags of every row
            const u64 *src = d.pair + (int64_t)par * n;
            u64 w[NU];
            uint32_t polls = 0u;
            for (;;) {
                bool ready = true;
#pragma unroll
                for (int u = 0; u < NU; ++u) {
                    const int k = tid + u * RT;
                    if (k < n) w[u] = ld_dev(src, (uint32_t)k);
                }
#pragma unroll
                for (int u = 0; u < NU; ++u)
                    if (tid + u * RT < n) ready &= (uint32_t)(w[u] >> 33) == (uint32_t)(t + 1);
                if (ready) break;
                if (++polls > *L.limit) {
                    *L.fail = 1;
                    break;
                }
            }
            uint32_t enow = 0u;
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                const int k = tid + u * RT;
                if (k < n) {
                    L.t[k] = __uint_as_float((uint32_t)w[u]);
                    enow |= (uint32_t)((w[u] >> 32) & 1ull) << u;
                } else if (k < NC) {
                    L.t[k] = 0.0f;         // (the reduction's scratch was here)
                }
            }
            if (enow != eprev) L.cnt[nu] = 1;      // (every writer writes 1)
            eprev = enow;
        } else {
            const int lr = tid;
            uint32_t enow = 0u;
            __syncthreads();
            if (lr < rows) enow = (uint32_t)L.e[lr];
            if (enow != eprev) L.cnt[nu] = 1;
            eprev = enow;
        }
        if (tid == 0) {
            L.cnt[nu ^ 1] = 0;
            if (M > 1 && t == *L.give_up) *L.fail = 1;
            if (first) *L.limit = kPollLimit;
        }
        __syncthreads();
        if (*L.fail) return false;
        // the set of iteration t (none at t = 0) against the one before
        if (!first) run = (t > 1 && !L.cnt[nu]) ? run + 1 : 1;
    }

    // ---- R_T, A_T.  From here on a wait given up leaves messages that are no
    // start any more, and says so (wrote).  One given up above does not: a
    // member that writes waits below for the flags of all, so where one has
    // left the loop early, every member that wrote gives up there.
    __syncthreads();
#pragma unroll
    for (int q = 0; q < RPW; ++q) {
        const int lr = wave + q * RW, i = row0 + lr;
        if (lr >= rows) continue;
        const int64_t at = (int64_t)i * d.ld;
#pragma unroll
        for (int j = 0; j < EJ; ++j) {
            const int c = 4 * (64 * j + lane);
            if (c >= n) continue;
            v4f ro, ao;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                ro[e] = c + e == i ? rd[q] : r[q][j][e];
                ao[e] = c + e == i ? ad[q] : a[q][j][e];
            }
            if (c + 3 < n) {
                st_row(d.R + at + c, ro);
                st_row(d.A + at + c, ao);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (c + e < n) {
                        st_one(d.R + at + c + e, ro[e]);
                        st_one(d.A + at + c + e, ao[e]);
                    }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    }

    // ---- labels: every member needs the whole exemplar set (a mask 0 / -inf
    // over the columns, in the place of t)
    const uint32_t fin = (uint32_t)t + 2u;       // stamps above every iteration's
    if (M > 1) {
        u64 *flags = d.pair + 2 * (int64_t)n;
        if (tid < rows) st_dev(flags + row0 + tid, ((u64)fin << 32) | (u64)L.e[tid]);
        for (int k = tid; k < n; k += RT) {
            u64 w;
            uint32_t polls = 0u;
            while ((uint32_t)((w = ld_dev(flags + k)) >> 32) != fin)
                if (++polls > kPollLimit) {
                    *L.fail = 1;
                    break;
                }
            L.t[k] = (w & 1ull) ? 0.0f : kNegInf;
        }
    } else {
        for (int k = tid; k < n; k += RT) L.t[k] = L.e[k] ? 0.0f : kNegInf;
    }
    for (int k = n + tid; k < NC; k += RT) L.t[k] = kNegInf;
    if (M > 1 && *L.give_up == kGiveUpAtEnd) *L.fail = 1;
    __syncthreads();
    if (*L.fail) {
        if (tid == 0) d.out->wrote = 1;
        return false;
    }
    u64 *con = d.pair + 3 * (int64_t)n;
#pragma unroll
    for (int q = 0; q < RPW; ++q) {
        const int lr = wave + q * RW, i = row0 + lr;
        if (lr >= rows) continue;
        float best = kNegInf;
        int at = INT32_MAX;
#pragma unroll
        for (int j = 0; j < EJ; ++j) {
            const float4 mv = *reinterpret_cast<const float4 *>(L.t + 4 * (64 * j + lane));
            const float m4[4] = {mv.x, mv.y, mv.z, mv.w};
            const v4f s4 = get_s(q, lr, j);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                // (an exemplar at -inf counts too: the lowest one, where no other is nearer)
                const int k = 4 * (64 * j + lane) + e;
                if (m4[e] == 0.0f && (s4[e] > best || (s4[e] == best && k < at))) {
                    best = s4[e];
                    at = k;
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int o = 32; o >= 1; o >>= 1) {
            const float ov = __shfl_xor(best, o, 64);
            const int ok = __shfl_xor(at, o, 64);
            if (ov > best || (ov == best && ok < at)) {
                best = ov;
                at = ok;
            }
        }
        if (lane == 0) {
            const int is = L.e[lr];
            const int lab = is ? i : at == INT32_MAX ? -1 : at;
            d.idx[i] = lab;
            d.eflag[i] = (uint8_t)is;
            // kind of contribution: 1 exemplar, 2 member of a class, 0 none
            const uint32_t kind = is ? 1u : lab >= 0 ? 2u : 0u;
            st_dev(con + i, ((u64)((fin << 2) | kind) << 32) | __float_as_uint(is ? sd[q] : best));
        }
    }
    if (rank != 0) return true;
    // ---- dpsim and expref (FP64, 1024 strided sums, then a tree), |E|
    double *sh = reinterpret_cast<double *>(L.pos);   // (and L.s: the labels have been taken)
    __syncthreads();
    int nex = 0;
    for (int x = tid; x < 1024; x += RT) {
        double s0 = 0.0, s1 = 0.0;
        for (int k = x; k < n; k += 1024) {
            u64 w;
            uint32_t polls = 0u;
            while ((uint32_t)((w = ld_dev(con + k)) >> 34) != fin)
                if (++polls > kPollLimit) {
                    *L.fail = 1;
                    break;
                }
            const uint32_t kind = (uint32_t)(w >> 32) & 3u;
            const double v = (double)__uint_as_float((uint32_t)w);
            s0 += kind == 2u ? v : 0.0;
            s1 += kind == 1u ? v : 0.0;
            nex += kind == 1u;
        }
        sh[x] = s0;
        sh[1024 + x] = s1;
    }
    if (tid == 0) L.cnt[0] = 0;
    __syncthreads();
    if (nex) atomicAdd(&L.cnt[0], nex);
    for (int w = 512; w >= 1; w >>= 1) {
        if (tid < w) {
            sh[tid] += sh[tid + w];
            sh[1024 + tid] += sh[1024 + tid + w];
        }
        __syncthreads();
    }
    if (*L.fail) {
        if (tid == 0) d.out->wrote = 1;
        return false;
    }
    if (tid == 0) {
        ResOut o;
        o.dpsim = sh[0];
        o.expref = sh[1024];
        o.iterations = t;
        o.converged = converged;
        o.n_exemplars = L.cnt[0];
        o.done = 1;
        o.wrote = 1;
        o.pad = 0;
        *d.out = o;
    }
    return true;
}

// A value that is the same in all lanes, in scalar registers (a batch reads its
// tables with vector loads: the rows need those registers).
template <class V>
__device__ __forceinline__ V scalar(const V &x) {
    struct Words {
        int w[sizeof(V) / 4];
    };
    static_assert(sizeof(Words) == sizeof(V), "whole words");
    Words a = __builtin_bit_cast(Words, x);
#pragma unroll
    for (int i = 0; i < (int)(sizeof(V) / 4); ++i) a.w[i] = __builtin_amdgcn_readfirstlane(a.w[i]);
    return __builtin_bit_cast(V, a);
}

template <int EJ, int RPW>
__global__ __launch_bounds__(RT) void k_resident(ResArgs p) {
    extern __shared__ char lds[];
    (void)res_run<EJ, RPW>(p.one, blockIdx.x, p, lds);
}

// Waits until every member of the instance has come to it (the others may
// still be at work on earlier instances, for as long as those run), or until
// a wait has been given up somewhere.
__device__ __forceinline__ bool all_arrived(const ResInst &d, int rank, const u64 *abort, char *lds) {
    int *stop = reinterpret_cast<int *>(lds);
    if (threadIdx.x == 0) {
        *stop = 0;
        st_dev(d.stat + rank, ~0ull);
    }
    __syncthreads();
    if ((int)threadIdx.x < d.members) {
        uint32_t polls = 0u;
        while (ld_dev(d.stat + threadIdx.x) == 0ull) {
            __builtin_amdgcn_s_sleep(8);
            if (ld_dev(abort) != 0ull || ++polls > kArriveLimit) {
                *stop = 1;
                break;
            }
        }
    }
    __syncthreads();
    const bool ok = *stop == 0;
    __syncthreads();
    return ok;
}

// True when every workgroup of the grid runs: from then on a wait between
// them ends.  Otherwise nothing has been started, and nothing is.
__device__ __forceinline__ bool grid_met(const ResArgs &p, char *lds) {
    int *stop = reinterpret_cast<int *>(lds);
    if (threadIdx.x == 0) {
        *stop = 0;
        atomicAdd(p.abort + 1, 1ull);
        uint32_t polls = 0u;
        while (p.give_up == 0 || ld_dev(p.abort + 1) < (u64)gridDim.x) {
            __builtin_amdgcn_s_sleep(8);
            if (p.give_up == 0 || ld_dev(p.abort) != 0ull || ++polls > kMeetLimit) {
                st_dev(p.abort, 1ull);
                *stop = 1;
                break;
            }
        }
    }
    __syncthreads();
    const bool ok = *stop == 0;
    __syncthreads();
    return ok;
}

// Many instances of uneven size: workgroup b runs its tasks in turn.  The
// tasks of every workgroup are in one order of the instances, so the first
// instance not yet done always has all of its members at work on it.
template <int CLASS>
__global__ __launch_bounds__(RT) void k_resident_batch(ResArgs p) {
    extern __shared__ char lds[];
    const int q1 = p.lane[blockIdx.x + 1];
    if (!grid_met(p, lds)) return;
    for (int q = p.lane[blockIdx.x]; q < q1; ++q) {
        const ResTask tk = scalar(p.tasks[q]);
        const ResInst d = scalar(p.insts[tk.inst]);
        bool ok = false;
        if (d.members > 1 && !all_arrived(d, tk.rank, p.abort, lds)) return;
#define APX_RES_CASE(e, w) case e * 16 + w: ok = res_run<e, w>(d, tk.rank, p, lds); break;
        if constexpr (CLASS == 0) {
            switch (d.variant) {
                APX_RES_CLASS0(APX_RES_CASE)
            default: break;
            }
        } else if constexpr (CLASS == 1) {
            switch (d.variant) {
                APX_RES_CLASS1(APX_RES_CASE)
            default: break;
            }
        } else {
            switch (d.variant) {
                APX_RES_CLASS2(APX_RES_CASE)
            default: break;
            }
        }
#undef APX_RES_CASE
        if (!ok) {
            if (threadIdx.x == 0) st_dev(p.abort, 1ull);
            return;
        }
        __syncthreads();
    }
}

// Admission of launches whose workgroups wait for each other to the compute
// units of a device, in order of arrival.
struct CuGate {
    std::mutex m;
    std::condition_variable cv;
    uint64_t next = 0, serving = 0;
    int used = 0;
    std::atomic<int> contexts{0};
};
constexpr int kGates = 64;
CuGate &gate_of(int device) {
    static CuGate *const gates = new CuGate[kGates];    // (never destroyed: threads may outlive main)
    return gates[device & (kGates - 1)];
}

// Zeroes the exchange words (8 bytes each) of the instance.
__global__ __launch_bounds__(256) void k_res_zero(u64 *p, int64_t words) {
    for (int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x; i < words; i += (int64_t)gridDim.x * 256) p[i] = 0ull;
}

constexpr int kMinPos = 2 * 1024 * 8;   // the final sums' scratch, in the place of max(0, r)

size_t res_lds(int ej, int rows) {
    const size_t nc = 256 * (size_t)ej;
    const size_t tw = nc * 4 > RT * 8 ? nc * 4 : RT * 8;
    const size_t part = 256 * (size_t)((ej + res_parts(ej) - 1) / res_parts(ej));
    const size_t pos = (size_t)rows * 4 * (part + 256 * (size_t)res_s_chunks(ej));
    return tw + 3 * 4 * kMaxRows + 32 + (pos > kMinPos ? pos : kMinPos);
}

}  // namespace

bool res_plan(int64_t n, int num_cus, int max_rows, ResPlan *pl) {
    if (n < 2 || n > kResMaxN) return false;
    ResPlan p{};
    p.ej = (int)((n + 255) / 256);
    p.groups = n <= 512 ? (int)n : 512;
    // as many whole groups per member as max_rows hold
    int rows = 0;
    for (p.gpm = (int)((int64_t)max_rows * p.groups / n); p.gpm >= 1; --p.gpm) {
        p.members = (p.groups + p.gpm - 1) / p.gpm;
        rows = 0;
        for (int m = 0; m < p.members; ++m) {
            const int a = m * p.gpm, b = a + p.gpm < p.groups ? a + p.gpm : p.groups;
            const int r = (int)((int64_t)b * n / p.groups - (int64_t)a * n / p.groups);
            rows = r > rows ? r : rows;
        }
        if (rows <= max_rows) break;
    }
    if (p.gpm < 1 || p.members > num_cus) return false;
    p.rows = rows;
    // the smallest instantiated number of rows per wavefront that holds them
    p.rpw = 0;
#define APX_RES_PICK(e, w) if (p.ej == e && w * RW >= rows && (p.rpw == 0 || w < p.rpw)) p.rpw = w;
    APX_RES_VARIANTS(APX_RES_PICK)
#undef APX_RES_PICK
    if (p.rpw == 0 || rows > kMaxRows) return false;
    p.lds = res_lds(p.ej, rows);
    p.words = 2 * n * p.members + 4 * n + p.members;
    *pl = p;
    return true;
}

void res_exchange(const ResPlan &pl, int64_t n, void *mem, ResInst *d) {
    unsigned long long *w = static_cast<unsigned long long *>(mem);
    d->members = pl.members;
    d->groups = pl.groups;
    d->gpm = pl.gpm;
    d->variant = pl.ej * 16 + pl.rpw;
    d->part = w;
    d->pair = w + 2 * n * pl.members;
    d->stat = d->pair + 4 * n;
}

hipError_t launch_res_zero(void *mem, int64_t words, hipStream_t s) {
    const int64_t want = (words + 255) / 256;
    k_res_zero<<<(unsigned)(want < 2048 ? want : 2048), 256, 0, s>>>(static_cast<unsigned long long *>(mem), words);
    return hipGetLastError();
}

int res_max_rows(int64_t n) {
    const int ej = (int)((n + 255) / 256);
    int most = 0;
#define APX_RES_MOST(e, w) if (ej == e && w > most) most = w;
    APX_RES_VARIANTS(APX_RES_MOST)
#undef APX_RES_MOST
    return most * RW;
}

int res_class(int64_t n) { return (int)((n - 1) / (256 * kClassChunks)); }
static_assert(kResMaxN == kResClasses * 256 * kClassChunks, "classes");

hipError_t launch_resident_batch(int cls, int grid, size_t lds, const ResInst *insts, const ResTask *tasks,
                                 const int32_t *lane, unsigned long long *abort, float lam, int32_t max_iter,
                                 int32_t conv_iter, int32_t give_up, hipStream_t s) {
    ResArgs a{};
    a.give_up = give_up;
    a.insts = insts;
    a.tasks = tasks;
    a.lane = lane;
    a.abort = abort;
    a.lam = a.lam0 = lam;
    a.max_iter = max_iter;
    a.conv_iter = conv_iter;
    // (a plain launch; see CuHold)
    const void *f = cls == 0   ? reinterpret_cast<const void *>(&k_resident_batch<0>)
                    : cls == 1 ? reinterpret_cast<const void *>(&k_resident_batch<1>)
                               : reinterpret_cast<const void *>(&k_resident_batch<2>);
    hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    void *args[] = {&a};
    return hipLaunchKernel(f, dim3(grid), dim3(RT), args, (unsigned)lds, s);
}

hipError_t launch_resident(const ResPlan &pl, const ResInst &d, float lam, float lam0, int32_t max_iter,
                           int32_t conv_iter, int32_t give_up, hipStream_t s) {
    ResArgs a{};
    a.give_up = give_up;
    a.one = d;
    a.lam = lam;
    a.lam0 = lam0;
    a.max_iter = max_iter;
    a.conv_iter = conv_iter;
    const void *f = nullptr;
    switch (d.variant) {
#define APX_RES_CASE(e, w) case e * 16 + w: f = reinterpret_cast<const void *>(&k_resident<e, w>); break;
        APX_RES_VARIANTS(APX_RES_CASE)
#undef APX_RES_CASE
    default: return hipErrorInvalidValue;
    }
    hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)pl.lds);
    if (e != hipSuccess) return e;
    void *args[] = {&a};
    return hipLaunchKernel(f, dim3(pl.members), dim3(RT), args, (unsigned)pl.lds, s);
}

void cu_contexts(int device, int change) { gate_of(device).contexts += change; }

CuHold::CuHold(int device, hipStream_t s, int workgroups, int num_cus) : device(device) {
    CuGate &g = gate_of(device);
    // Work the stream still has to do is not waited for inside the gate,
    // where it would keep out other contexts.
    if (g.contexts > 1 && hipStreamQuery(s) == hipErrorNotReady) (void)hipStreamSynchronize(s);
    units = (workgroups + 7) & ~7;
    std::unique_lock<std::mutex> l(g.m);
    const uint64_t mine = g.next++;
    g.cv.wait(l, [&] { return mine == g.serving && (g.used == 0 || g.used + units <= num_cus); });
    ++g.serving;
    g.used += units;
    l.unlock();
    g.cv.notify_all();
}

CuHold::~CuHold() {
    CuGate &g = gate_of(device);
    {
        std::lock_guard<std::mutex> l(g.m);
        g.used -= units;
    }
    g.cv.notify_all();
}

}  // namespace apx
