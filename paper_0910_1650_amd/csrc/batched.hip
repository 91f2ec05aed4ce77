// batched.hip -- many independent AP instances of uneven size at once
// (Algorithm 1 run on each instance; the sub-problems of partition AP,
// Algorithm 2 Step 2, are such a batch).
//
// Instances of up to kResMaxN points go to the one-launch solve with messages
// in registers (resident.hip): 64 instances of 100 to 1000 points (64-D) take
// 3.2 ms so, 37 ms in the streaming launch below, whose teams flush the L2s
// four times per iteration at their barriers.  The streaming launch keeps the
// larger instances.  It is a fixed grid of workgroups that are all resident at once (a
// cooperative launch).  The host cuts the grid into teams over a ragged
// table: an instance gets a team of g workgroups in proportion to its n^2
// (member r owns a contiguous block of rows and the same block of columns
// for the column sums), or, when there are more instances than workgroups,
// one-workgroup teams each solve a queue of instances in turn.  A team runs
// its instance from the prologue to the instance's own stop rule on the
// device: per iteration a row pass (A_t, decisions, R_{t+1}, column
// partials), a team barrier, the column sums of the member's columns in
// FP64 in a fixed order and the stop rule (member 0), a team barrier.  The
// host waits for the one launch; no iteration is driven from the host.
#include <algorithm>
#include <chrono>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "apx_internal.h"

namespace apx {
namespace {

constexpr float kNegInf = -INFINITY;
constexpr int BT = 256;   // threads per work item

struct InstDesc {
    const float *S;
    float *R[2];          // R_t lives in R[t & 1]
    float *A;
    int64_t ld;
    int32_t n;
    int32_t nparts;       // team size (= partial rows) of this instance
    float *partial;       // [nparts][ldp]
    int64_t ldp;
    float *tcol, *ccol, *rdiag;
    uint8_t *eflag;
    int32_t *dec;
    ApState *st;
    int32_t *idx;         // labels (caller's)
    int32_t *ex;          // exemplar list scratch (n)
    double *sums;         // [dpsim, expref]
    int32_t *nex_out;
    int32_t pad;
};

__device__ __forceinline__ float f4get(const float4 &v, int e) {
    return e == 0 ? v.x : e == 1 ? v.y : e == 2 ? v.z : v.w;
}
__device__ __forceinline__ void f4set(float4 &v, int e, float x) {
    if (e == 0) v.x = x;
    else if (e == 1) v.y = x;
    else if (e == 2) v.z = x;
    else v.w = x;
}

__device__ __forceinline__ void top2_merge(float &v1, int &k1, float &v2, float ov1, int ok1, float ov2) {
    const bool take = (ov1 > v1) || (ov1 == v1 && ok1 < k1);
    const float nv2 = take ? fmaxf(ov2, v1) : fmaxf(v2, ov1);
    v1 = take ? ov1 : v1;
    k1 = take ? ok1 : k1;
    v2 = nv2;
}
__device__ __forceinline__ void argmax_merge(float &v, int &k, float ov, int ok) {
    const bool take = ov > v || (ov == v && ok < k);
    v = take ? ov : v;
    k = take ? ok : k;
}

// Rows [row0, row1) of one instance: same arithmetic as the single-instance
// pass (Eqs. (2)-(4) with damping, decision, column partials into partial
// row `part`).  MODE: PASS_FULL, PASS_R_ONLY, PASS_R_COLD (also writes
// A_0 = 0).  sh_f / sh_i: the workgroup's reduction slots.
template <int J, int MODE>
__device__ __forceinline__ void rows_pass(const InstDesc *dp, int row0, int row1, int part, float lam, int32_t t,
                                          float (*sh_f)[BT / 64][3], int (*sh_i)[BT / 64][2]) {
#pragma clang fp contract(off)
    const InstDesc d = *dp;
    constexpr bool DO_A = (MODE == PASS_FULL);
    constexpr bool LD_RA = (MODE != PASS_R_COLD);
    constexpr int NW = BT / 64;

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int n = d.n;
    const int64_t ld = d.ld;
    const float oml = 1.0f - lam;
    // (selects, not an index: an indexed member would put d in scratch)
    const float *Rin = (t & 1) ? d.R[1] : d.R[0];
    float *Rout = (t & 1) ? d.R[0] : d.R[1];
    const float4 z4 = make_float4(0.f, 0.f, 0.f, 0.f);

    float4 part4[J];
#pragma unroll
    for (int j = 0; j < J; ++j) part4[j] = z4;
    int my_nex = 0, my_changed = 0;

    for (int i = row0; i < row1; ++i) {
        const float *Srow = d.S + (int64_t)i * ld;
        const float *Rrow = Rin + (int64_t)i * ld;
        float *Arow = d.A + (int64_t)i * ld;
        float *Orow = Rout + (int64_t)i * ld;
        const float ci = DO_A ? d.ccol[i] : 0.0f;
        float v1 = kNegInf, v2 = kNegInf, dv = kNegInf;
        int k1 = INT32_MAX, dk = INT32_MAX;
        float4 u[J];
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int c = (j * BT + tid) * 4;
            u[j] = z4;
            if (c >= n) continue;
            const bool full = c + 3 < n;
            const float4 s4 = *reinterpret_cast<const float4 *>(Srow + c);
            float4 r4 = z4, a4 = z4;
            if constexpr (LD_RA) {
                r4 = *reinterpret_cast<const float4 *>(Rrow + c);
                a4 = *reinterpret_cast<const float4 *>(Arow + c);
            }
            float4 t4 = z4;
            if constexpr (DO_A) t4 = *reinterpret_cast<const float4 *>(d.tcol + c);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int k = c + e;
                if (!(full || k < n)) continue;
                float a = f4get(a4, e);
                const float r = f4get(r4, e);
                if constexpr (DO_A) {
                    const float upd = (k == i) ? ci : fminf(0.0f, f4get(t4, e) - fmaxf(0.0f, r));
                    a = lam * a + oml * upd;
                    f4set(a4, e, a);
                    const float dvv = a + r;
                    const bool gt = dvv > dv;
                    dk = gt ? k : dk;
                    dv = gt ? dvv : dv;
                }
                const float v = a + f4get(s4, e);
                const bool gt = v > v1;
                v2 = gt ? v1 : fmaxf(v2, v);
                k1 = gt ? k : k1;
                v1 = gt ? v : v1;
                f4set(u[j], e, lam * r + oml * f4get(s4, e));
            }
            if constexpr (DO_A || MODE == PASS_R_COLD) {
                if (full) {
                    *reinterpret_cast<float4 *>(Arow + c) = a4;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (c + e < n) Arow[c + e] = f4get(a4, e);
                }
            }
        }
        // workgroup reduction (wavefront butterflies, then across wavefronts)
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            top2_merge(v1, k1, v2, __shfl_xor(v1, off, 64), __shfl_xor(k1, off, 64),
                       __shfl_xor(v2, off, 64));
            if constexpr (DO_A) argmax_merge(dv, dk, __shfl_xor(dv, off, 64), __shfl_xor(dk, off, 64));
        }
        const int slot = i & 1;
        if (lane == 0) {
            sh_f[slot][wave][0] = v1;
            sh_f[slot][wave][1] = v2;
            sh_f[slot][wave][2] = dv;
            sh_i[slot][wave][0] = k1;
            sh_i[slot][wave][1] = dk;
        }
        __syncthreads();
        v1 = sh_f[slot][0][0];
        v2 = sh_f[slot][0][1];
        dv = sh_f[slot][0][2];
        k1 = sh_i[slot][0][0];
        dk = sh_i[slot][0][1];
#pragma unroll
        for (int w = 1; w < NW; ++w) {
            top2_merge(v1, k1, v2, sh_f[slot][w][0], sh_i[slot][w][0], sh_f[slot][w][1]);
            if constexpr (DO_A) argmax_merge(dv, dk, sh_f[slot][w][2], sh_i[slot][w][1]);
        }
        if constexpr (DO_A) {
            if (tid == 0) {
                d.dec[i] = dk;
                const uint8_t e = (uint8_t)(dk == i);
                if (d.eflag[i] != e) my_changed = 1;
                d.eflag[i] = e;
                my_nex += e;
            }
        }
        const float m_other = oml * v1, m_self = oml * v2;
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int c = (j * BT + tid) * 4;
            if (c >= n) continue;
            const bool full = c + 3 < n;
            float4 rn;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int k = c + e;
                const float v = f4get(u[j], e) - (k == k1 ? m_self : m_other);
                f4set(rn, e, v);
                if (k < n) {
                    if (k == i) d.rdiag[i] = v;
                    else f4set(part4[j], e, f4get(part4[j], e) + fmaxf(0.0f, v));
                }
            }
            if (full) {
                *reinterpret_cast<float4 *>(Orow + c) = rn;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (c + e < n) Orow[c + e] = f4get(rn, e);
            }
        }
    }
    float *P = d.partial + (int64_t)part * d.ldp;
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int c = (j * BT + tid) * 4;
        if (c < n) *reinterpret_cast<float4 *>(P + c) = part4[j];
    }
    if constexpr (DO_A) {
        if (tid == 0) {
            if (my_nex) atomicAdd(&d.st->nex, my_nex);
            if (my_changed) atomicOr(&d.st->changed, 1);
        }
    }
}

// Column sums of columns [c0, c1) of one instance over its nparts partial
// rows, in FP64: 16 columns at a time, 16 slices of the partial rows per
// column, slices combined in a fixed order (deterministic).
__device__ __forceinline__ void col_sums(const InstDesc *dp, int c0, int c1, double (*red)[16]) {
#pragma clang fp contract(off)
    const InstDesc d = *dp;
    const int cx = threadIdx.x & 15, sl = threadIdx.x >> 4;
    for (int cb = c0; cb < c1; cb += 16) {
        const int k = cb + cx;
        double c = 0.0;
        if (k < c1) {
            int g = sl;
            for (; g + 3 * 16 < d.nparts; g += 4 * 16) {
                float v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = d.partial[(int64_t)(g + u * 16) * d.ldp + k];
#pragma unroll
                for (int u = 0; u < 4; ++u) c += (double)v[u];
            }
            for (; g < d.nparts; g += 16) c += (double)d.partial[(int64_t)g * d.ldp + k];
        }
        red[sl][cx] = c;
        __syncthreads();
        if (sl == 0 && k < c1) {
            double tot = 0.0;
#pragma unroll
            for (int q = 0; q < 16; ++q) tot += red[q][cx];
            d.tcol[k] = (float)((double)d.rdiag[k] + tot);
            d.ccol[k] = (float)tot;
        }
        __syncthreads();
    }
}

// The stop rule of one instance after the pass of iteration st->iter + 1
// (the exemplar-set rule and the iteration cap).
__device__ __forceinline__ void bookkeep(ApState *st) {
    const int t = st->iter + 1;
    const int same = (t > 1) && (st->changed == 0);
    const int run = same ? st->run + 1 : 1;
    st->iter = t;
    st->run = run;
    st->last_nex = st->nex;
    if (st->conv_iter > 0 && run >= st->conv_iter && st->nex > 0) {
        st->converged = 1;
        st->frozen = 1;
    } else if (t >= st->max_iter) {
        st->frozen = 1;
    }
    st->nex = 0;
    st->changed = 0;
}

// Barrier of a team of g workgroups (g > 1): arrival counter and generation
// word; the last to arrive resets the counter and publishes the next
// generation.  Writes before the barrier are released at device scope and
// acquired after it.  The wait is bounded: after about kSpinLimit polls
// (seconds; a legitimate wait is one member's row pass, well under a
// millisecond) the fail flag is raised and the workgroup gives up, so a
// broken team cannot hang the device; the host reports the failure.
struct TeamBar {
    uint32_t count;
    uint32_t gen;
    uint32_t pad[62];    // one 256-byte line per team
};
constexpr uint32_t kSpinLimit = 1u << 22;

// Returns false (in every thread) when the team has failed.
__device__ __forceinline__ bool team_sync(TeamBar *bar, int g, uint32_t &gen, int32_t *fail, int *ok_sh) {
    if (g == 1) {
        __syncthreads();
        return true;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        __threadfence();
        const uint32_t target = gen + 1u;
        if (atomicAdd(&bar->count, 1u) == (uint32_t)g - 1u) {
            atomicExch(&bar->count, 0u);
            __threadfence();
            atomicExch(&bar->gen, target);
        } else {
            uint32_t spins = 0;
            while (__hip_atomic_load(&bar->gen, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_AGENT) != target) {
                __builtin_amdgcn_s_sleep(4);
                if (++spins > kSpinLimit) {
                    atomicOr(fail, 1);
                    break;
                }
            }
        }
        __threadfence();
        gen = target;
        *ok_sh = __hip_atomic_load(fail, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == 0;
    }
    __syncthreads();
    return *ok_sh != 0;
}

// One task: instance `inst`, member `rank` of a team of g workgroups (team
// barrier `bar`, -1 for a team of one).
struct Task {
    int32_t inst, rank, g, bar;
};

struct PersistArgs {
    const InstDesc *descs;
    const Task *tasks;
    const int32_t *lane;      // workgroup b runs tasks [lane[b], lane[b+1]) in order
    TeamBar *bars;
    int32_t *fail;
    float lam;
    int32_t warm;
};

// The whole batched solve in one launch: every workgroup runs its tasks in
// turn; a task is Algorithm 1 on one instance, from the prologue (R_1) to
// the instance's own stop rule, in lockstep with the rest of its team.
// The shortest rows keep four workgroups per compute unit (128 registers);
// longer rows take the registers their chunks need (the occupancy query
// sets the grid).
template <int J>
__global__ __launch_bounds__(BT, J <= 1 ? 4 : 1) void k_batch_persist(PersistArgs a) {
    __shared__ float sh_f[2][BT / 64][3];
    __shared__ int sh_i[2][BT / 64][2];
    __shared__ double red[16][16];
    __shared__ int ok_sh, frozen_sh;
    const int b = blockIdx.x;
    for (int q = a.lane[b]; q < a.lane[b + 1]; ++q) {
        const Task tk = a.tasks[q];
        const InstDesc *d = a.descs + tk.inst;
        ApState *st = d->st;
        TeamBar *bar = tk.bar >= 0 ? a.bars + tk.bar : nullptr;
        uint32_t gen = 0u;
        const int n = d->n;
        const int row0 = (int)((int64_t)tk.rank * n / tk.g);
        const int row1 = (int)((int64_t)(tk.rank + 1) * n / tk.g);
        // t = 0: R_1 from R_0 (zero, or given) and A_0 (zero: written here)
        if (a.warm == APX_COLD) rows_pass<J, PASS_R_COLD>(d, row0, row1, tk.rank, a.lam, 0, sh_f, sh_i);
        else rows_pass<J, PASS_R_ONLY>(d, row0, row1, tk.rank, a.lam, 0, sh_f, sh_i);
        if (!team_sync(bar, tk.g, gen, a.fail, &ok_sh)) return;
        col_sums(d, row0, row1, red);
        if (!team_sync(bar, tk.g, gen, a.fail, &ok_sh)) return;
        for (int32_t t = 1;; ++t) {
            rows_pass<J, PASS_FULL>(d, row0, row1, tk.rank, a.lam, t, sh_f, sh_i);
            if (!team_sync(bar, tk.g, gen, a.fail, &ok_sh)) return;
            col_sums(d, row0, row1, red);
            if (tk.rank == 0 && threadIdx.x == 0) bookkeep(st);
            if (!team_sync(bar, tk.g, gen, a.fail, &ok_sh)) return;
            if (threadIdx.x == 0) frozen_sh = __hip_atomic_load(&st->frozen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            __syncthreads();
            const int fz = frozen_sh;
            __syncthreads();
            if (fz) break;
        }
    }
}

__global__ void k_batch_init(const InstDesc *descs, int count, int32_t max_iter, int32_t conv_iter) {
    const int j = blockIdx.x;
    if (j >= count) return;
    const InstDesc d = descs[j];
    if (threadIdx.x == 0) {
        ApState s{};
        s.max_iter = max_iter;
        s.conv_iter = conv_iter;
        *d.st = s;
    }
    for (int i = threadIdx.x; i < d.n; i += blockDim.x) d.eflag[i] = 0;
}

// R_T into the caller's buffer when T is odd (R_T then lives in R[1]).
__global__ void k_batch_fix_r(const InstDesc *descs) {
    const InstDesc d = descs[blockIdx.y];
    if ((d.st->iter & 1) == 0) return;
    for (int64_t i = blockIdx.x; i < d.n; i += gridDim.x) {
        const float *src = d.R[1] + i * d.ld;
        float *dst = d.R[0] + i * d.ld;
        for (int c = threadIdx.x; c < d.n; c += blockDim.x) dst[c] = src[c];
    }
}

// Zero A (A_0 = 0) or R (R_0 = 0) of every instance.
__global__ void k_batch_zero(const InstDesc *descs, int which) {
    const InstDesc d = descs[blockIdx.y];
    float *M = which == 0 ? d.A : d.R[0];
    for (int64_t i = blockIdx.x; i < d.n; i += gridDim.x)
        for (int c = threadIdx.x; c < d.n; c += blockDim.x) M[i * d.ld + c] = 0.0f;
}

// Labels and FP64 net similarity, one workgroup per instance: exemplar list
// (ascending), then each non-exemplar takes the exemplar of largest s(i,k)
// (lowest k on ties); sums formed in a fixed order.
__global__ __launch_bounds__(1024) void k_batch_finalize(const InstDesc *descs) {
    const InstDesc d = descs[blockIdx.x];
    __shared__ int wcount[16];
    __shared__ int base;
    __shared__ double red[2][1024];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) base = 0;
    __syncthreads();
    for (int k0 = 0; k0 < d.n; k0 += 1024) {
        const int k = k0 + tid;
        const bool e = (k < d.n) && d.eflag[k];
        const unsigned long long m = __ballot(e);
        const int before = __popcll(m & ((1ull << lane) - 1ull));
        if (lane == 0) wcount[wave] = __popcll(m);
        __syncthreads();
        int off = base;
        for (int w = 0; w < wave; ++w) off += wcount[w];
        if (e) d.ex[off + before] = k;
        __syncthreads();
        if (tid == 0) {
            int tot = 0;
            for (int w = 0; w < 16; ++w) tot += wcount[w];
            base += tot;
        }
        __syncthreads();
    }
    const int m = base;
    double dp = 0.0, ep = 0.0;
    // one wavefront per row
    for (int i = wave; i < d.n; i += 16) {
        const float *Srow = d.S + (int64_t)i * d.ld;
        int lab;
        if (m == 0) {
            lab = -1;
        } else if (d.eflag[i]) {
            lab = i;
            if (lane == 0) ep += (double)Srow[i];
        } else {
            float bv = kNegInf;
            int bk = INT32_MAX;
            for (int j = lane; j < m; j += 64) {
                const int k = d.ex[j];
                const float v = Srow[k];
                if (v > bv || (v == bv && k < bk)) {
                    bv = v;
                    bk = k;
                }
            }
            for (int o = 32; o >= 1; o >>= 1) {
                const float ov = __shfl_xor(bv, o, 64);
                const int ok = __shfl_xor(bk, o, 64);
                if (ov > bv || (ov == bv && ok < bk)) {
                    bv = ov;
                    bk = ok;
                }
            }
            lab = bk;
            if (lane == 0) dp += (double)bv;
        }
        if (lane == 0) d.idx[i] = lab;
    }
    red[0][tid] = dp;
    red[1][tid] = ep;
    __syncthreads();
    for (int w = 512; w >= 1; w >>= 1) {
        if (tid < w) {
            red[0][tid] += red[0][tid + w];
            red[1][tid] += red[1][tid + w];
        }
        __syncthreads();
    }
    if (tid == 0) {
        d.sums[0] = red[0][0];
        d.sums[1] = red[1][0];
        *d.nex_out = m;
    }
}

template <int J>
hipError_t launch_persist(const PersistArgs &a, int grid, hipStream_t s) {
    void *args[] = {const_cast<PersistArgs *>(&a)};
    return hipLaunchCooperativeKernel(reinterpret_cast<const void *>(&k_batch_persist<J>), dim3(grid), dim3(BT),
                                      args, 0, s);
}

template <int J>
int persist_occupancy() {
    int nb = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_batch_persist<J>, BT, 0) != hipSuccess) nb = 0;
    return nb;
}

#define APX_BATCH_J(X) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12)

hipError_t persist_launch(int J, const PersistArgs &a, int grid, hipStream_t s) {
    switch (J) {
#define APX_CASE(j) case j: return launch_persist<j>(a, grid, s);
        APX_BATCH_J(APX_CASE)
#undef APX_CASE
    default: return hipErrorInvalidValue;
    }
}

int occupancy_of(int J) {
    switch (J) {
#define APX_CASE(j) case j: return persist_occupancy<j>();
        APX_BATCH_J(APX_CASE)
#undef APX_CASE
    default: return 0;
    }
}

}  // namespace

namespace {

// Workgroups per compute unit of the persistent launch (at most; fewer when
// the kernel's occupancy is lower), and the fewest rows a team member
// takes (a row costs a few microseconds of latency; two team barriers per
// iteration cost about as much as a few rows).  APX_BATCH_WPC and
// APX_BATCH_MIN_ROWS override them (tuning runs).
constexpr int kMaxWpc = 4;
constexpr int kMinMemberRows = 8;

int bit_length(int64_t v) {
    int b = 0;
    while (v > 0) {
        ++b;
        v >>= 1;
    }
    return b;
}

const BatchTune *find_batch_tune(const apx_ctx *ctx, int32_t count, int64_t max_n) {
    const int cb = bit_length(count), nb = bit_length(max_n);
    for (const BatchTune &t : ctx->btune)
        if (t.count_bits == cb && t.n_bits == nb) return &t;
    return nullptr;
}

int env_int(const char *name, int dflt, int lo, int hi) {
    const char *v = getenv(name);
    if (!v || !v[0]) return dflt;
    const int x = atoi(v);
    return x < lo ? lo : (x > hi ? hi : x);
}

struct BatchPlan {
    int J, wpc, G;
    std::vector<Task> tasks;
    std::vector<int32_t> lane;     // G + 1 entries
    std::vector<int32_t> team;     // team size per instance
    int nbars;
    // workspace offsets (relative to the plan's base)
    std::vector<size_t> o_r2, o_part, o_t, o_c, o_d, o_e, o_dec, o_ex;
    size_t o_st, o_sum, o_nex, o_desc, o_tasks, o_lane, o_bars, o_fail, bytes;
};

// Teams: with no more instances than workgroups, each instance gets its own
// team, sized in proportion to its n^2 (at least one workgroup, and no
// member with fewer than kMinMemberRows rows unless the team is one
// workgroup), scaled so the teams fill
// the grid; all instances then run at once.  With more instances than
// workgroups, every team is one workgroup and the instances are dealt to
// the workgroups largest first, each to the least loaded one.
BatchPlan make_plan(int32_t count, const BatchSpec *spec, int num_cus, int wpc, int min_rows) {
    BatchPlan P;
    int64_t max_n = 0;
    for (int j = 0; j < count; ++j) max_n = spec[j].n > max_n ? spec[j].n : max_n;
    P.J = (int)((max_n + 4 * BT - 1) / (4 * BT));
    P.wpc = wpc;
    P.G = num_cus * wpc;
    const int G = P.G;
    P.team.assign(count, 1);
    P.lane.assign(G + 1, 0);
    std::vector<double> cost(count);
    double tot = 0.0;
    for (int j = 0; j < count; ++j) {
        cost[j] = (double)spec[j].n * (double)spec[j].n;
        tot += cost[j];
    }
    std::vector<std::vector<Task>> per(G);
    P.nbars = 0;
    if (count <= G) {
        auto gmax = [&](int j) -> int64_t {
            const int64_t m = spec[j].n / min_rows;
            return m < 1 ? 1 : m;
        };
        auto sizes = [&](double x, std::vector<int32_t> &g) -> int64_t {
            int64_t sum = 0;
            for (int j = 0; j < count; ++j) {
                int64_t v = (int64_t)(x * cost[j] / tot);
                const int64_t m = gmax(j);
                v = v < 1 ? 1 : (v > m ? m : v);
                g[j] = (int32_t)v;
                sum += v;
            }
            return sum;
        };
        std::vector<int32_t> g(count);
        double lo = 0.0, hi = (double)G;
        while (sizes(hi, g) <= G && hi < 1e12) hi *= 2.0;
        for (int it = 0; it < 60; ++it) {
            const double mid = 0.5 * (lo + hi);
            if (sizes(mid, g) <= G) lo = mid;
            else hi = mid;
        }
        sizes(lo, g);
        int b = 0;
        for (int j = 0; j < count; ++j) {
            P.team[j] = g[j];
            const int bar = g[j] > 1 ? P.nbars++ : -1;
            for (int r = 0; r < g[j]; ++r) per[b++].push_back(Task{j, r, g[j], bar});
        }
    } else {
        std::vector<int> order(count);
        for (int j = 0; j < count; ++j) order[j] = j;
        std::stable_sort(order.begin(), order.end(), [&](int x, int y) { return cost[x] > cost[y]; });
        std::vector<double> load(G, 0.0);
        for (int j : order) {
            int best = 0;
            for (int b = 1; b < G; ++b)
                if (load[b] < load[best]) best = b;
            load[best] += cost[j];
            per[best].push_back(Task{j, 0, 1, -1});
        }
    }
    for (int b = 0; b < G; ++b) {
        P.lane[b] = (int32_t)P.tasks.size();
        P.tasks.insert(P.tasks.end(), per[b].begin(), per[b].end());
    }
    P.lane[G] = (int32_t)P.tasks.size();

    WsLayout L;
    P.o_r2.resize(count); P.o_part.resize(count); P.o_t.resize(count); P.o_c.resize(count);
    P.o_d.resize(count); P.o_e.resize(count); P.o_dec.resize(count); P.o_ex.resize(count);
    for (int j = 0; j < count; ++j) {
        const int64_t n = spec[j].n, ldp = (n + 3) & ~int64_t(3);
        P.o_r2[j] = L.take(sizeof(float) * (size_t)n * (size_t)spec[j].ld);
        P.o_part[j] = L.take(sizeof(float) * (size_t)ldp * (size_t)P.team[j]);
        P.o_t[j] = L.take(sizeof(float) * ldp);
        P.o_c[j] = L.take(sizeof(float) * ldp);
        P.o_d[j] = L.take(sizeof(float) * ldp);
        P.o_e[j] = L.take((size_t)n);
        P.o_dec[j] = L.take(sizeof(int32_t) * n);
        P.o_ex[j] = L.take(sizeof(int32_t) * n);
    }
    P.o_st = L.take(sizeof(ApState) * count);
    P.o_sum = L.take(sizeof(double) * 2 * count);
    P.o_nex = L.take(sizeof(int32_t) * count);
    P.o_desc = L.take(sizeof(InstDesc) * count);
    P.o_tasks = L.take(sizeof(Task) * (P.tasks.size() > 0 ? P.tasks.size() : 1));
    P.o_lane = L.take(sizeof(int32_t) * (size_t)(G + 1));
    P.o_bars = L.take(sizeof(TeamBar) * (size_t)(P.nbars > 0 ? P.nbars : 1));
    P.o_fail = L.take(sizeof(int32_t));
    P.bytes = L.off;
    return P;
}

}  // namespace

namespace {

// Instances of up to kResMaxN points: the one-launch solve with messages in
// registers (resident.hip), many instances to a launch.
struct ResBatch {
    std::vector<int32_t> order;    // instances, largest first
    std::vector<ResPlan> plan;     // by position in `order`
    std::vector<ResTask> tasks;
    std::vector<int32_t> lane;     // grid + 1 entries
    std::vector<size_t> o_x, o_e;  // exchange words (relative to o_x0), flags
    int cls = 0;                   // res_class of all of them
    int grid = 0;
    size_t lds = 0;
    size_t o_tab, tab_bytes, o_task, o_lane, o_x0, x_bytes, o_out, o_abort, bytes;
};

// Few rows per member where the members of all instances then fit the chip
// at once (an iteration is four microseconds of exchange and 0.6 per chunk
// of four columns and row of a wavefront); else the most rows a member can
// hold, so that the instances take the fewest turns.
bool res_batch_plan(const BatchSpec *spec, const std::vector<int32_t> &order, int num_cus, ResBatch *B) {
    if (order.empty()) return false;
    B->cls = res_class(spec[order[0]].n);
    B->order = order;
    B->plan.resize(order.size());
    for (int rpw = 1; rpw <= 8; ++rpw) {
        const int lv = rpw * kResWaves;
        int64_t sum = 0;
        for (size_t q = 0; q < order.size(); ++q) {
            const int64_t n = spec[order[q]].n;
            const int most = res_max_rows(n);
            if (!res_plan(n, num_cus, lv < most ? lv : most, &B->plan[q]) &&
                !res_plan(n, num_cus, most, &B->plan[q]))
                return false;
            sum += B->plan[q].members;
        }
        if (sum <= num_cus) break;
    }
    // each instance, largest first, to the workgroups that are free soonest
    std::vector<std::pair<float, int>> load(num_cus);
    for (int b = 0; b < num_cus; ++b) load[b] = {0.0f, b};
    std::vector<std::vector<ResTask>> per(num_cus);
    for (size_t q = 0; q < order.size(); ++q) {
        const ResPlan &p = B->plan[q];
        if (p.members < num_cus) std::nth_element(load.begin(), load.begin() + p.members, load.end());
        float start = 0.0f;
        for (int m = 0; m < p.members; ++m) start = load[m].first > start ? load[m].first : start;
        const float end = start + 4.0f + 0.6f * (float)(p.ej * p.rpw);
        for (int m = 0; m < p.members; ++m) {
            load[m].first = end;
            per[load[m].second].push_back(ResTask{(int32_t)q, m});
        }
        B->lds = p.lds > B->lds ? p.lds : B->lds;
    }
    B->lane.push_back(0);
    for (int b = 0; b < num_cus; ++b)
        if (!per[b].empty()) {
            B->tasks.insert(B->tasks.end(), per[b].begin(), per[b].end());
            B->lane.push_back((int32_t)B->tasks.size());
            ++B->grid;
        }
    WsLayout L;
    B->o_tab = L.take(sizeof(ResInst) * order.size());
    B->o_task = L.take(sizeof(ResTask) * B->tasks.size());
    B->o_lane = L.take(sizeof(int32_t) * B->lane.size());
    B->tab_bytes = L.off;
    B->o_out = L.take(sizeof(ResOut) * order.size());
    B->o_abort = L.take(16);
    B->o_x0 = L.off;
    for (const ResPlan &p : B->plan) B->o_x.push_back(L.take(8 * (size_t)p.words));
    B->x_bytes = L.off - B->o_x0;
    for (int32_t j : order) B->o_e.push_back(L.take((size_t)spec[j].n));
    B->bytes = L.off;
    return true;
}

// The instances of one class of sizes, largest first.
std::vector<int32_t> res_order(int32_t count, const BatchSpec *spec, int cls) {
    std::vector<int32_t> order;
    for (int32_t j = 0; j < count; ++j)
        if (spec[j].n <= kResMaxN && res_class(spec[j].n) == cls) order.push_back(j);
    std::stable_sort(order.begin(), order.end(), [&](int32_t x, int32_t y) { return spec[x].n > spec[y].n; });
    return order;
}

// Solves the instances of the plan; results by instance number, done[j] set
// for those that ran to their end.  The others can run elsewhere: their
// workgroups gave up waiting for each other and left R and A as they were (or
// the start is cold).
apx_status res_batch_solve(apx_ctx *ctx, const ResBatch &B, const BatchSpec *spec, int32_t warm,
                           const apx_params *params, apx_result *res, char *done) {
    hipStream_t s = ctx->stream;
    char *b = static_cast<char *>(ctx->ws) + ctx->ws_base;
    const size_t cnt = B.order.size();
    std::vector<char> tab(B.tab_bytes, 0);
    ResInst *inst = reinterpret_cast<ResInst *>(tab.data() + B.o_tab);
    for (size_t q = 0; q < cnt; ++q) {
        const BatchSpec &sp = spec[B.order[q]];
        ResInst &d = inst[q];
        d.S = sp.S;
        d.R = sp.R;
        d.A = sp.A;
        d.ld = sp.ld;
        d.n = (int32_t)sp.n;
        d.load_a = warm != APX_COLD;
        d.load_r = warm == APX_WARM_AR;
        d.idx = sp.idx;
        d.eflag = reinterpret_cast<uint8_t *>(b + B.o_e[q]);
        d.out = reinterpret_cast<ResOut *>(b + B.o_out) + q;
        res_exchange(B.plan[q], sp.n, b + B.o_x[q], &d);
    }
    std::memcpy(tab.data() + B.o_task, B.tasks.data(), sizeof(ResTask) * B.tasks.size());
    std::memcpy(tab.data() + B.o_lane, B.lane.data(), sizeof(int32_t) * B.lane.size());
    // the results and the exchange words start at zero
    hipError_t e;
    std::vector<ResOut> out(cnt);
    const CuHold hold(ctx->device, s, B.grid, ctx->num_cus);
    if ((e = hipMemcpyAsync(b, tab.data(), B.tab_bytes, hipMemcpyHostToDevice, s)) ||
        (e = launch_res_zero(b + B.o_out, (int64_t)((B.o_x0 - B.o_out + B.x_bytes) / 8), s)) ||
        (e = launch_resident_batch(B.cls, B.grid, B.lds, reinterpret_cast<const ResInst *>(b + B.o_tab),
                                   reinterpret_cast<const ResTask *>(b + B.o_task),
                                   reinterpret_cast<const int32_t *>(b + B.o_lane),
                                   reinterpret_cast<unsigned long long *>(b + B.o_abort), params->damping,
                                   params->max_iter, params->conv_iter, ctx->give_up, s)) ||
        (e = hipMemcpyAsync(out.data(), b + B.o_out, sizeof(ResOut) * cnt, hipMemcpyDeviceToHost, s)) ||
        (e = hipStreamSynchronize(s)))
        return hip_err(ctx, e, "batched launch");
    for (size_t q = 0; q < cnt; ++q) {
        const ResOut &o = out[q];
        if (o.done != 1) {
            if (o.wrote && warm != APX_COLD)
                return set_err(ctx, APX_EDEVICE, "batched launch: a wait between workgroups timed out");
            continue;
        }
        done[B.order[q]] = 1;
        apx_result &r = res[B.order[q]];
        std::memset(&r, 0, sizeof r);
        r.iterations = o.iterations;
        r.converged = o.converged;
        r.n_exemplars = o.n_exemplars;
        if (o.n_exemplars == 0) {
            r.dpsim = r.expref = r.netsim = NAN;
        } else {
            r.dpsim = o.dpsim;
            r.expref = o.expref;
            r.netsim = o.dpsim + o.expref;
        }
        r.status = APX_OK;
    }
    return APX_OK;
}

}  // namespace

size_t batched_ws_bytes(int32_t count, const BatchSpec *spec, int num_cus) {
    // an upper bound: the streaming plan at the largest workgroups per CU and
    // the largest teams (one row per member at least), of all instances and of
    // those the other launches leave (fewer instances get larger teams)
    size_t bytes = make_plan(count, spec, num_cus, kMaxWpc, 1).bytes;
    std::vector<BatchSpec> rest;
    for (int32_t j = 0; j < count; ++j)
        if (spec[j].n > kResMaxN) rest.push_back(spec[j]);
    if (!rest.empty() && (int32_t)rest.size() < count) {
        const size_t r = make_plan((int32_t)rest.size(), rest.data(), num_cus, kMaxWpc, 1).bytes;
        bytes = r > bytes ? r : bytes;
    }
    for (int c = 0; c < kResClasses; ++c) {
        ResBatch B;
        if (res_batch_plan(spec, res_order(count, spec, c), num_cus, &B) && B.bytes > bytes) bytes = B.bytes;
    }
    return bytes;
}

namespace {
// The plan of the streaming batch, its workspace reserved: tuned for this batch
// shape if known (apx_autotune_batched), the environment (APX_BATCH_WPC,
// APX_BATCH_MIN_ROWS) over that, the tuner's candidate while it times.  A
// workspace that cannot grow (the caller's, or one with data of the running
// call below ws_base) gets smaller teams where it does not hold the plan's.
apx_status stream_plan(apx_ctx *ctx, int32_t count, const BatchSpec *spec, BatchPlan *P) {
    int64_t max_n = 0;
    for (int j = 0; j < count; ++j) max_n = spec[j].n > max_n ? spec[j].n : max_n;
    const int J = (int)((max_n + 4 * BT - 1) / (4 * BT));
    if (J > 12) return set_err(ctx, APX_ENOTIMPL, "batched instances are limited to n <= %d", 12 * 4 * BT);
    int wpc = occupancy_of(J);
    if (wpc < 1) return set_err(ctx, APX_EDEVICE, "no occupancy for the batched kernel");
    int cap = kMaxWpc, min_rows = kMinMemberRows;
    const BatchTune *bt = find_batch_tune(ctx, count, max_n);
    if (bt) {
        cap = bt->wpc;
        min_rows = bt->min_rows;
    }
    cap = env_int("APX_BATCH_WPC", cap, 1, kMaxWpc);
    min_rows = env_int("APX_BATCH_MIN_ROWS", min_rows, 1, 1 << 20);
    if (ctx->force_bwpc) cap = ctx->force_bwpc;
    if (ctx->force_bmin) min_rows = ctx->force_bmin;
    wpc = wpc < cap ? wpc : cap;
    *P = make_plan(count, spec, ctx->num_cus, wpc, min_rows);
    const bool fixed = ctx->ws_external || ctx->ws_base > 0;
    while (fixed && ctx->ws_base + P->bytes > ctx->ws_bytes && min_rows < max_n) {
        min_rows *= 4;
        *P = make_plan(count, spec, ctx->num_cus, wpc, min_rows);
    }
    return ws_reserve(ctx, ctx->ws_base + P->bytes);
}

// The streaming batch: tables, initial state, one persistent cooperative
// launch, then R_T and the labels.
apx_status batched_stream(apx_ctx *ctx, int32_t count, const BatchSpec *spec, int32_t warm, const apx_params *params,
                          apx_result *res);
}  // namespace

// Host driver shared by ap_solve_batched and pap_solve (Step 2): the
// workspace slice starts at ctx->ws_base.
apx_status batched_solve(apx_ctx *ctx, int32_t count, const BatchSpec *spec, int32_t warm,
                         const apx_params *params, apx_result *res) {
    int64_t max_n = 0;
    for (int j = 0; j < count; ++j) max_n = spec[j].n > max_n ? spec[j].n : max_n;
    if (max_n > 12 * 4 * BT)
        return set_err(ctx, APX_ENOTIMPL, "batched instances are limited to n <= %d", 12 * 4 * BT);
    // Instances whose messages fit in registers go first, one launch for each
    // class of sizes; a forced or hand-set plan of the launch below (the tuner,
    // APX_BATCH_WPC, APX_BATCH_MIN_ROWS) keeps every instance there, and so
    // does a workspace without room for theirs.
    const bool streamed = ctx->force_bwpc || ctx->force_bmin || getenv("APX_BATCH_WPC") || getenv("APX_BATCH_MIN_ROWS");
    const bool fixed = ctx->ws_external || ctx->ws_base > 0;
    ctx->last_fallback = 0;
    std::vector<char> done(count, 0);
    ResBatch cls[kResClasses];
    bool use[kResClasses];
    for (int c = 0; c < kResClasses; ++c) {
        use[c] = !streamed && res_batch_plan(spec, res_order(count, spec, c), ctx->num_cus, &cls[c]) &&
                 !(fixed && ctx->ws_base + cls[c].bytes > ctx->ws_bytes);
        if (use[c])
            for (int32_t j : cls[c].order) done[j] = 1;
    }
    std::vector<int32_t> left;
    std::vector<BatchSpec> rest;
    auto collect = [&]() {
        left.clear();
        rest.clear();
        for (int32_t j = 0; j < count; ++j)
            if (!done[j]) {
                left.push_back(j);
                rest.push_back(spec[j]);
            }
    };
    // Room for all that will run is found before anything does: a call that
    // does not fit leaves every output as it was.
    collect();
    if (!rest.empty()) {
        BatchPlan P;
        const apx_status st = stream_plan(ctx, (int32_t)rest.size(), rest.data(), &P);
        if (st != APX_OK) return st;
    }
    for (int c = 0; c < kResClasses; ++c)
        if (use[c]) {
            const apx_status st = ws_reserve(ctx, ctx->ws_base + cls[c].bytes);
            if (st != APX_OK) return st;
        }
    for (int c = kResClasses - 1; c >= 0; --c) {
        if (!use[c]) continue;
        for (int32_t j : cls[c].order) done[j] = 0;
        const apx_status st = res_batch_solve(ctx, cls[c], spec, warm, params, res, done.data());
        if (st != APX_OK) return st;
        for (int32_t j : cls[c].order)
            if (!done[j]) ctx->last_fallback = APX_FALLBACK_WAIT;
    }
    collect();
    if (rest.empty()) return APX_OK;
    std::vector<apx_result> rr(rest.size());
    const apx_status st = batched_stream(ctx, (int32_t)rest.size(), rest.data(), warm, params, rr.data());
    if (st == APX_OK)
        for (size_t q = 0; q < left.size(); ++q) res[left[q]] = rr[q];
    return st;
}

namespace {
apx_status batched_stream(apx_ctx *ctx, int32_t count, const BatchSpec *spec, int32_t warm, const apx_params *params,
                          apx_result *res) {
    hipStream_t s = ctx->stream;
    int64_t max_n = 0;
    for (int j = 0; j < count; ++j) max_n = spec[j].n > max_n ? spec[j].n : max_n;
    const int J = (int)((max_n + 4 * BT - 1) / (4 * BT));
    BatchPlan P;
    const apx_status st = stream_plan(ctx, count, spec, &P);
    if (st != APX_OK) return st;
    char *b = static_cast<char *>(ctx->ws) + ctx->ws_base;

    ApState *dst = reinterpret_cast<ApState *>(b + P.o_st);
    double *dsum = reinterpret_cast<double *>(b + P.o_sum);
    int32_t *dnex = reinterpret_cast<int32_t *>(b + P.o_nex);
    std::vector<InstDesc> descs(count);
    for (int j = 0; j < count; ++j) {
        InstDesc &d = descs[j];
        std::memset(&d, 0, sizeof d);
        d.S = spec[j].S;
        d.R[0] = spec[j].R;
        d.R[1] = reinterpret_cast<float *>(b + P.o_r2[j]);
        d.A = spec[j].A;
        d.ld = spec[j].ld;
        d.n = (int32_t)spec[j].n;
        d.nparts = P.team[j];
        d.partial = reinterpret_cast<float *>(b + P.o_part[j]);
        d.ldp = (spec[j].n + 3) & ~int64_t(3);
        d.tcol = reinterpret_cast<float *>(b + P.o_t[j]);
        d.ccol = reinterpret_cast<float *>(b + P.o_c[j]);
        d.rdiag = reinterpret_cast<float *>(b + P.o_d[j]);
        d.eflag = reinterpret_cast<uint8_t *>(b + P.o_e[j]);
        d.dec = reinterpret_cast<int32_t *>(b + P.o_dec[j]);
        d.st = dst + j;
        d.idx = spec[j].idx;
        d.ex = reinterpret_cast<int32_t *>(b + P.o_ex[j]);
        d.sums = dsum + 2 * j;
        d.nex_out = dnex + j;
    }
    InstDesc *ddesc = reinterpret_cast<InstDesc *>(b + P.o_desc);
    Task *dtasks = reinterpret_cast<Task *>(b + P.o_tasks);
    int32_t *dlane = reinterpret_cast<int32_t *>(b + P.o_lane);
    TeamBar *dbars = reinterpret_cast<TeamBar *>(b + P.o_bars);
    int32_t *dfail = reinterpret_cast<int32_t *>(b + P.o_fail);
    hipError_t e;
    if ((e = hipMemcpyAsync(ddesc, descs.data(), sizeof(InstDesc) * count, hipMemcpyHostToDevice, s)) ||
        (!P.tasks.empty() &&
         (e = hipMemcpyAsync(dtasks, P.tasks.data(), sizeof(Task) * P.tasks.size(), hipMemcpyHostToDevice, s))) ||
        (e = hipMemcpyAsync(dlane, P.lane.data(), sizeof(int32_t) * P.lane.size(), hipMemcpyHostToDevice, s)) ||
        (e = hipStreamSynchronize(s)))
        return hip_err(ctx, e, "batch tables");

    const dim3 zgrid((unsigned)(max_n < 2048 ? max_n : 2048), (unsigned)count);
    k_batch_init<<<count, 256, 0, s>>>(ddesc, count, params->max_iter, params->conv_iter);
    if ((e = hipGetLastError())) return hip_err(ctx, e, "batch init");
    // team barriers and the fail flag start at zero (a fill kernel, not a memset)
    if ((e = launch_fill_u8(reinterpret_cast<uint8_t *>(dbars), sizeof(TeamBar) * (P.nbars > 0 ? P.nbars : 1), 0, s)) ||
        (e = launch_fill_u8(reinterpret_cast<uint8_t *>(dfail), sizeof(int32_t), 0, s)))
        return hip_err(ctx, e, "batch barriers");
    if (warm == APX_WARM_A) {
        k_batch_zero<<<zgrid, 256, 0, s>>>(ddesc, 1);
        if ((e = hipGetLastError())) return hip_err(ctx, e, "R_0");
    }
    // (as many workgroups as fit: the whole chip)
    const CuHold hold(ctx->device, s, ctx->num_cus, ctx->num_cus);
    PersistArgs pa{ddesc, dtasks, dlane, dbars, dfail, params->damping, warm};
    if ((e = persist_launch(J, pa, P.G, s))) return hip_err(ctx, e, "persistent batch launch");
    k_batch_fix_r<<<zgrid, 256, 0, s>>>(ddesc);
    if ((e = hipGetLastError())) return hip_err(ctx, e, "copy R");
    k_batch_finalize<<<count, 1024, 0, s>>>(ddesc);
    if ((e = hipGetLastError())) return hip_err(ctx, e, "finalize");
    std::vector<ApState> hst(count);
    std::vector<double> sums(2 * (size_t)count);
    std::vector<int32_t> nex(count);
    int32_t hfail = 0;
    if ((e = hipMemcpyAsync(hst.data(), dst, sizeof(ApState) * count, hipMemcpyDeviceToHost, s)) ||
        (e = hipMemcpyAsync(sums.data(), dsum, sizeof(double) * 2 * count, hipMemcpyDeviceToHost, s)) ||
        (e = hipMemcpyAsync(nex.data(), dnex, sizeof(int32_t) * count, hipMemcpyDeviceToHost, s)) ||
        (e = hipMemcpyAsync(&hfail, dfail, sizeof(int32_t), hipMemcpyDeviceToHost, s)) ||
        (e = hipStreamSynchronize(s)))
        return hip_err(ctx, e, "results");
    if (hfail) return set_err(ctx, APX_EDEVICE, "batched launch: a team barrier timed out");
    for (int j = 0; j < count; ++j) {
        apx_result &r = res[j];
        std::memset(&r, 0, sizeof r);
        r.iterations = hst[j].iter;
        r.converged = hst[j].converged;
        r.n_exemplars = nex[j];
        if (nex[j] == 0) {
            r.dpsim = r.expref = r.netsim = NAN;
        } else {
            r.dpsim = sums[2 * j];
            r.expref = sums[2 * j + 1];
            r.netsim = r.dpsim + r.expref;
        }
        r.status = APX_OK;
    }
    return APX_OK;
}
}  // namespace

}  // namespace apx

// ---- tuning of the batched plan --------------------------------------------
using namespace apx;

namespace {

// Deterministic finite scratch similarities in [-1, 0) (a small integer hash
// per element, the diagonal at -1/2): the batch timing runs a fixed number
// of iterations, so only the shapes matter.
__global__ void k_btune_fill(float *S, int64_t n, int64_t ld, uint32_t salt) {
    for (int64_t i = blockIdx.x; i < n; i += gridDim.x)
        for (int64_t k = threadIdx.x; k < n; k += blockDim.x) {
            const uint32_t h = ((uint32_t)i * 2654435761u) ^ ((uint32_t)k * 40503u) ^ (salt * 97u);
            S[i * ld + k] = i == k ? -0.5f : -(float)((h >> 7) & 1023u) / 1024.0f - 1.0f / 2048.0f;
        }
}

}  // namespace

extern "C" apx_status apx_autotune_batched(apx_ctx *ctx, int32_t count, const int64_t *sizes, int32_t *wpc_out,
                                           int32_t *min_rows_out, double *ms_out) {
    if (!ctx) return APX_EINVAL;
    if (count < 1 || !sizes) return set_err(ctx, APX_EINVAL, "need count >= 1 and sizes");
    // A call with this batch streams the instances above kResMaxN, and looks a
    // plan up for those: they are what is timed.  Without one the plan is that
    // of the whole batch, for when all of it streams.
    std::vector<int64_t> streamed;
    for (int j = 0; j < count; ++j) {
        if (sizes[j] < 2 || sizes[j] > 12 * 4 * BT)
            return set_err(ctx, APX_EINVAL, "instance %d: need 2 <= n <= %d", j, 12 * 4 * BT);
        if (sizes[j] > kResMaxN) streamed.push_back(sizes[j]);
    }
    if (!streamed.empty()) {
        sizes = streamed.data();
        count = (int32_t)streamed.size();
    }
    int64_t max_n = 0, total = 0;
    std::vector<int64_t> lds(count), offs(count);
    for (int j = 0; j < count; ++j) {
        const int64_t n = sizes[j];
        max_n = n > max_n ? n : max_n;
        lds[j] = (n + 3) & ~int64_t(3);
        offs[j] = total;
        total += n * lds[j];
    }
    int cur = -1;
    (void)hipGetDevice(&cur);
    if (cur != ctx->device) (void)hipSetDevice(ctx->device);
    hipStream_t s = ctx->stream;
    // S, R, A of every instance in one buffer, labels in another
    float *buf = nullptr;
    int32_t *lab = nullptr;
    struct Free {
        float **b;
        int32_t **l;
        ~Free() {
            if (*b) (void)hipFree(*b);
            if (*l) (void)hipFree(*l);
        }
    } fr{&buf, &lab};
    hipError_t e;
    if ((e = hipMalloc(&buf, sizeof(float) * 3 * (size_t)total)) ||
        (e = hipMalloc(&lab, sizeof(int32_t) * (size_t)count * (size_t)max_n)))
        return hip_err(ctx, e, "batch tuning scratch");
    std::vector<BatchSpec> spec(count);
    for (int j = 0; j < count; ++j) {
        float *Sj = buf + offs[j];
        spec[j] = BatchSpec{sizes[j], lds[j], Sj, buf + total + offs[j], buf + 2 * total + offs[j], lab + (size_t)j * max_n};
        const int g = (int)(sizes[j] < 1024 ? sizes[j] : 1024);
        k_btune_fill<<<g, 256, 0, s>>>(Sj, sizes[j], lds[j], (uint32_t)j);
    }
    if ((e = hipGetLastError())) return hip_err(ctx, e, "batch tuning fill");
    apx_params p{};
    p.damping = 0.9f;
    p.max_iter = 12;
    p.conv_iter = 0;
    std::vector<apx_result> res(count);
    const int J = (int)((max_n + 4 * BT - 1) / (4 * BT));
    int occ = occupancy_of(J);
    occ = occ < kMaxWpc ? occ : kMaxWpc;
    if (occ < 1) return set_err(ctx, APX_EDEVICE, "no occupancy for the batched kernel");
    const int rows_c[3] = {2, 8, 32};
    double best = 1e300;
    int bw = 0, bm = 0;
    auto timed = [&](int w, int m, double *ms) -> apx_status {
        ctx->force_bwpc = w;
        ctx->force_bmin = m;
        ctx->ws_base = 0;
        const auto t0 = std::chrono::steady_clock::now();
        const apx_status st = batched_solve(ctx, count, spec.data(), APX_COLD, &p, res.data());
        *ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
        ctx->force_bwpc = ctx->force_bmin = 0;
        return st;
    };
    double ms = 0.0;
    apx_status st = timed(occ, kMinMemberRows, &ms);   // warm-up (module load, workspace)
    if (st != APX_OK) return st;
    for (int w = 1; w <= occ; ++w)
        for (int m : rows_c) {
            double t = 1e300;
            for (int rep = 0; rep < 2; ++rep) {
                st = timed(w, m, &ms);
                if (st != APX_OK) return st;
                t = ms < t ? ms : t;
            }
            if (t < best) {
                best = t;
                bw = w;
                bm = m;
            }
        }
    const BatchTune nt{bit_length(count), bit_length(max_n), bw, bm, best};
    bool put = false;
    for (BatchTune &t : ctx->btune)
        if (t.count_bits == nt.count_bits && t.n_bits == nt.n_bits) {
            t = nt;
            put = true;
        }
    if (!put) ctx->btune.push_back(nt);
    if (wpc_out) *wpc_out = bw;
    if (min_rows_out) *min_rows_out = bm;
    if (ms_out) *ms_out = best;
    return APX_OK;
}
